"""GPU parity of the 3 x 3 stride-2 weight gradient.  From an uncompressed record (tiles of one column), whose copy waves
split their registers differently: odd and even maps, rows of one to eight segments, ragged channels, tiles of 1 x 1
and 2 x 1.  From pooled records: every width of tile, which each have a kernel, with whole and with ragged tiles."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2409_11902_amd import binding as B
from paper_2409_11902_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    # name, N, C, K, H, W, kh, the split
    ("rows of two segments", 9, 70, 96, 28, 28, 1, 0),
    ("rows of four segments", 4, 64, 40, 30, 56, 1, 0),
    ("odd map", 7, 33, 65, 27, 15, 1, 0),
    ("one segment, several images per chunk", 31, 64, 128, 14, 14, 1, 0),
    ("tiny maps", 40, 20, 24, 5, 4, 1, 0),
    ("rows of eight segments", 40, 16, 32, 9, 120, 1, 1),
    ("tiles of two rows, one column", 6, 48, 64, 22, 26, 2, 0),
    ("many chunks, rows of two segments", 100, 70, 96, 28, 28, 1, 1),
    ("many chunks, rows of four segments", 64, 64, 40, 30, 56, 1, 1),
    ("many chunks, odd map", 430, 33, 65, 27, 15, 1, 1),
    ("many chunks, 64 x 64 tile", 300, 128, 260, 14, 14, 1, 1),
    ("many chunks, tiles of two rows, one column", 400, 48, 64, 22, 26, 2, 1),
    ("chunks of two rows instead of one, 16 Z items per thread", 40, 224, 272, 20, 56, 1, 2),
    ("the same in rows of odd length", 33, 210, 264, 21, 53, 1, 2),
    ("16 Z items per thread in the 32 x 32 tile", 133, 68, 66, 35, 60, 1, 2),
    ("the same in rows of odd length", 155, 68, 69, 27, 61, 1, 2),
    ("tiles of eight rows, one column: longer chunks without a split", 421, 33, 260, 18, 18, 8, 0),
]


def check(name, N, C, K, H, W, kh, kw, wide):
    import torch
    from gpu_util import Guarded, download, upload, workspace
    spec = synth.LayerSpec(name, N, C, K, H, W, stride=2)
    t = synth.make_inputs(spec, "dw-uncompressed-s2", tensors=("X", "dY"))
    d = B.desc_from_spec(spec, pool_kh=kh, pool_kw=kw)
    plan = B.cac_describe_plan(d, B.OP_BWD_WEIGHT_COMPRESSED)
    split = ("", "registers split towards Z (4 dY, 8 Z)", "registers split towards Z (2 dY, 16 Z)")[wide]
    assert plan.startswith("dw_mfma") and (split in plan if split else "registers split" not in plan), plan
    hp, wp, _, _ = B.cac_pooled_shape(d)
    Z, dW = Guarded((N, C, hp, wp), torch.bfloat16), Guarded((K, C, 3, 3), torch.float32)
    B.cac_compress(d, upload(t["X"], spec.dtype), Z.t)
    B.conv_bwd_weight_compressed(d, Z.t, upload(t["dY"], spec.dtype), dW.t, workspace(d, B.OP_BWD_WEIGHT_COMPRESSED))
    torch.cuda.synchronize()
    Z.check("Z"), dW.check("dW")
    g = oracle.ConvGeom(N, C, K, H, W, 3, 3, 2, 2, 1, 1)
    want = oracle.conv_dw(g, oracle.inflate(download(Z.t), H, W, kh, kw), t["dY"].astype(np.float64))
    # identical bfloat16 operands, exact products: only the order of at most N * P * Q float additions differs, about
    # sqrt(42140) * 2^-24 = 1.2e-5 of the result's norm; any wrong term is orders above
    for tap in range(9):
        w = want[:, :, tap // 3, tap % 3]
        assert np.linalg.norm(download(dW.t)[:, :, tap // 3, tap % 3] - w) <= 2e-5 * np.linalg.norm(w), (name, tap)


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_weight_gradient(case):
    name, N, C, K, H, W, kh, wide = case
    check(name, N, C, K, H, W, kh, 1, wide)


@pytest.mark.parametrize("kw", [2, 4, 8])
@pytest.mark.parametrize("shape", [(9, 33, 65, 27, 29), (300, 128, 260, 14, 16)], ids=["ragged, pixels over the waves", "64 x 64 tile"])
def test_weight_gradient_pooled(shape, kw):
    check(f"tiles of {kw} columns", *shape, kw, kw, 0)
