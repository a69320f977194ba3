"""The float convolution whose filter operands a lane reads as they lie (csrc/conv_lds.hip, 3 x 3 and 1 x 1, strides 1 and 2): parity
classes, channel counts past a multiple of 16 -- what follows a filter's row there is the next one, possibly infinite --, more
of a patch than is kept in registers, and four pixels per thread."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2409_11902_amd import binding as B
from paper_2409_11902_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    # name, N, C, K, H, W, R, stride, pad
    ("3x3 stride 2", 3, 21, 37, 13, 18, 3, 2, 1),
    ("3x3 stride 2, odd extents", 5, 33, 17, 15, 11, 3, 2, 1),
    ("1x1 stride 2", 4, 40, 23, 14, 9, 1, 2, 0),
    ("1x1", 3, 50, 35, 11, 13, 1, 1, 0),
    ("3x3 without padding", 2, 18, 31, 10, 12, 3, 1, 0),
    ("two columns of batches", 2, 35, 48, 9, 70, 3, 1, 1),
    ("more batches than registers", 1, 19, 33, 12, 200, 3, 1, 1),
    ("four pixels per thread", 40, 20, 35, 40, 52, 3, 1, 1),
    ("1x1, four pixels per thread", 80, 35, 53, 33, 52, 1, 1, 0),
]


@pytest.mark.parametrize("infinite", [False, True], ids=["finite", "infinite weight"])
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_forward_and_data_gradient(case, infinite):
    import torch
    from gpu_util import Guarded, download, upload
    name, N, C, K, H, W, R, st, pad = case
    d = B.make_desc(N, C, K, H, W, R, R, st, st, pad, pad, 1, 1, dtype=B.F32)
    assert all(B.cac_describe_plan(d, op).startswith("conv_lds") for op in (B.OP_FWD_AND_COMPRESS, B.OP_BWD_DATA))
    P, Q = B.cac_out_shape(d)
    rng = np.random.default_rng(sum(map(ord, name)))
    make = lambda *s: synth.to_storage(rng.standard_normal(s, dtype=np.float32), synth.F32)  # noqa: E731
    X, Wt, b, dY = make(N, C, H, W), make(K, C, R, R), make(K), make(N, K, P, Q)
    if infinite:
        Wt[2, 0, R // 2, 0], Wt[K - 1, 1, 0, R // 2] = np.inf, np.nan
    Y, Z, dX = (Guarded(s, torch.float32) for s in ((N, K, P, Q), (N, C, H, W), (N, C, H, W)))
    up = lambda a: upload(a, synth.F32)  # noqa: E731
    B.conv_fwd_and_compress(d, up(X), up(Wt), up(b), Y.t, Z.t)
    B.conv_bwd_data(d, up(Wt), up(dY), dX.t)
    torch.cuda.synchronize()
    g = oracle.ConvGeom(N, C, K, H, W, R, R, st, st, pad, pad)
    f = [a.astype(np.float64) for a in (X, Wt, b, dY)]
    # float sums of at most 9 * 67 terms of either sign: sqrt(603) * 2^-24 = 1.5e-6 of the result
    for what, out, want in (("Y", Y, oracle.conv_fwd(g, f[0], f[1], f[2])), ("dX", dX, oracle.conv_dx(g, f[1], f[3]))):
        out.check(what)
        got, ok = download(out.t), np.isfinite(want)
        assert ok.all() != infinite or what == "dX"
        assert np.array_equal(np.isfinite(got), ok), (name, what)
        assert np.linalg.norm(got[ok] - want[ok]) <= 1e-5 * np.linalg.norm(want[ok]), (name, what)
