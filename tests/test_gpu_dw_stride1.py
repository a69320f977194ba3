"""GPU parity of the 3 x 3 stride-1 weight gradient.  From an uncompressed record with the copy registers split towards Z: both
tiles, every row length that has a kernel, rows of odd length, a last chunk that is not full, rows that no other split takes.  From
pooled records: every width of tile, which each have a kernel, and chunks of whole images with a last one that is not full."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2409_11902_amd import binding as B
from paper_2409_11902_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    # name, N, C, K, H, W, kh, kw, tile, towards Z
    ("two segments", 2, 64, 65, 31, 14, 1, 1, 32, True),
    ("two segments, odd rows", 3, 300, 65, 31, 15, 1, 1, 32, True),
    ("four segments", 2, 64, 64, 31, 32, 1, 1, 32, True),
    ("four segments, odd rows", 7, 33, 65, 37, 31, 1, 1, 32, True),
    ("five segments, odd rows", 1, 64, 65, 38, 33, 1, 1, 32, True),
    ("seven segments", 1, 64, 64, 15, 56, 1, 1, 32, True),
    ("seven segments, odd rows", 5, 33, 40, 19, 55, 1, 1, 32, True),
    ("ten segments", 3, 64, 64, 14, 80, 1, 1, 32, True),
    ("rows that only this split takes", 2, 60, 70, 11, 112, 1, 1, 32, True),
    ("the same of odd length", 3, 33, 65, 13, 111, 1, 1, 32, True),
    ("one segment, 64 x 64 tile", 207, 100, 128, 37, 8, 2, 1, 64, True),
    ("one segment, odd rows, 64 x 64 tile", 169, 300, 40, 38, 7, 2, 1, 64, True),
    ("two segments, odd rows, 64 x 64 tile", 206, 130, 40, 23, 15, 1, 1, 64, True),
    ("four segments, 64 x 64 tile", 204, 33, 65, 37, 28, 1, 1, 64, True),
    ("five segments, odd rows, 64 x 64 tile", 175, 33, 65, 35, 33, 1, 1, 64, True),
    ("seven segments, 64 x 64 tile", 202, 33, 40, 30, 50, 2, 1, 64, True),
    ("whole images, the last chunk not full", 203, 260, 164, 4, 4, 2, 2, 32, False),
    ("whole images of odd rows, the last chunk not full", 123, 164, 260, 7, 7, 2, 2, 32, False),
    ("tiles of 4 columns, ragged", 9, 33, 65, 27, 29, 4, 4, 32, False),
    ("tiles of 8 columns, ragged", 9, 33, 65, 27, 29, 8, 8, 64, False),
    ("tiles of 8 columns, one segment", 9, 33, 65, 27, 8, 8, 8, 32, False),
    ("tiles of 8 columns, 64 x 64 tile", 300, 128, 260, 14, 16, 8, 8, 64, False),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_weight_gradient(case):
    import torch
    from gpu_util import Guarded, download, upload, workspace
    name, N, C, K, H, W, kh, kw, tile, split = case
    spec = synth.LayerSpec(name, N, C, K, H, W)
    t = synth.make_inputs(spec, "dw-stride1", tensors=("X", "dY"))
    d = B.desc_from_spec(spec, pool_kh=kh, pool_kw=kw)
    plan = B.cac_describe_plan(d, B.OP_BWD_WEIGHT_COMPRESSED)
    assert f"tile={tile}x{tile} " in plan and ("registers split towards Z (4 dY, 8 Z)" in plan) == split, plan
    hp, wp, _, _ = B.cac_pooled_shape(d)
    Z, dW = Guarded((N, C, hp, wp), torch.bfloat16), Guarded((K, C, 3, 3), torch.float32)
    B.cac_compress(d, upload(t["X"], spec.dtype), Z.t)
    B.conv_bwd_weight_compressed(d, Z.t, upload(t["dY"], spec.dtype), dW.t, workspace(d, B.OP_BWD_WEIGHT_COMPRESSED))
    torch.cuda.synchronize()
    Z.check("Z"), dW.check("dW")
    want = oracle.conv_dw(oracle.ConvGeom(N, C, K, H, W, 3, 3, 1, 1, 1, 1), oracle.inflate(download(Z.t), H, W, kh, kw), t["dY"].astype(np.float64))
    # identical bfloat16 operands, exact products: only the order of at most N * H * W float additions differs, about the root of
    # their number times 2^-24 of the result's norm; any wrong term is orders above
    tol = 2 * np.sqrt(N * H * W) * 2.0 ** -24
    for tap in range(9):
        w = want[:, :, tap // 3, tap % 3]
        assert np.linalg.norm(download(dW.t)[:, :, tap // 3, tap % 3] - w) <= tol * np.linalg.norm(w), (name, tap)
