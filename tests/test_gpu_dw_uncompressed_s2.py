"""GPU parity of the 3 x 3 stride-2 weight gradient from an uncompressed record (tiles of one column), whose copy waves
split their registers differently: odd and even maps, rows of one to eight segments, ragged channels, tiles of 1 x 1
and 2 x 1."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2409_11902_amd import binding as B
from paper_2409_11902_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    # name, N, C, K, H, W, kh
    ("rows of two segments", 9, 70, 96, 28, 28, 1),
    ("rows of four segments", 4, 64, 40, 30, 56, 1),
    ("odd map", 7, 33, 65, 27, 15, 1),
    ("one segment, several images per chunk", 31, 64, 128, 14, 14, 1),
    ("tiny maps", 40, 20, 24, 5, 4, 1),
    ("rows of eight segments", 2, 16, 32, 9, 120, 1),
    ("tiles of two rows, one column", 6, 48, 64, 22, 26, 2),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_weight_gradient(case):
    import torch
    from gpu_util import Guarded, download, upload, workspace
    name, N, C, K, H, W, kh = case
    spec = synth.LayerSpec(name, N, C, K, H, W, stride=2)
    t = synth.make_inputs(spec, "dw-uncompressed-s2", tensors=("X", "dY"))
    d = B.desc_from_spec(spec, pool_kh=kh, pool_kw=1)
    assert B.cac_describe_plan(d, B.OP_BWD_WEIGHT_COMPRESSED).startswith("dw_mfma")
    hp, wp, _, _ = B.cac_pooled_shape(d)
    Z, dW = Guarded((N, C, hp, wp), torch.bfloat16), Guarded((K, C, 3, 3), torch.float32)
    B.cac_compress(d, upload(t["X"], spec.dtype), Z.t)
    B.conv_bwd_weight_compressed(d, Z.t, upload(t["dY"], spec.dtype), dW.t, workspace(d, B.OP_BWD_WEIGHT_COMPRESSED))
    torch.cuda.synchronize()
    Z.check("Z"), dW.check("dW")
    g = oracle.ConvGeom(N, C, K, H, W, 3, 3, 2, 2, 1, 1)
    want = oracle.conv_dw(g, oracle.inflate(download(Z.t), H, W, kh, 1), t["dY"].astype(np.float64))
    # identical bfloat16 operands, exact products: only the order of at most N * P * Q float additions differs, about
    # sqrt(1800) * 2^-24 = 2.5e-6 of the result's norm; any wrong term is orders above
    for tap in range(9):
        w = want[:, :, tap // 3, tap % 3]
        assert np.linalg.norm(download(dW.t)[:, :, tap // 3, tap % 3] - w) <= 2e-5 * np.linalg.norm(w), (name, tap)
