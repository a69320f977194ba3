"""GPU parity of the LDS-tiled float forward / data-gradient kernel (conv_lds.hip) at the edges of what it takes:
one and four pixels per thread, rows that share a wave and rows longer than one, several images per workgroup,
channel counts around its blocks of 16 and 4, strides with pixels that no tap reaches, large filters, and shapes
that do not fit LDS (the plain kernels)."""
from __future__ import annotations

import re

import numpy as np
import pytest

import oracle
from paper_2409_11902_amd import binding as B
from paper_2409_11902_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    # name, dtype, N, C, K, H, W, R, S, stride_h, stride_w, pad_h, pad_w
    ("one pixel per thread", "f32", 3, 16, 16, 32, 32, 3, 3, 1, 1, 1, 1),
    ("four pixels per thread", "f32", 40, 20, 33, 40, 52, 3, 3, 1, 1, 1, 1),
    ("several images per workgroup", "f32", 37, 17, 15, 3, 5, 3, 3, 1, 1, 1, 1),
    ("one pixel images", "f32", 70, 5, 18, 1, 1, 1, 1, 1, 1, 0, 0),
    ("rows longer than a wave", "f32", 2, 9, 16, 6, 150, 3, 3, 1, 1, 1, 1),
    ("four channels per pass", "f32", 1, 11, 17, 5, 400, 3, 5, 1, 1, 1, 2),
    ("stride 3 past a 1x1 filter", "f32", 4, 16, 19, 13, 11, 1, 1, 3, 3, 0, 0),
    ("uneven strides and pads", "f32", 3, 18, 35, 17, 14, 3, 5, 2, 3, 2, 0),
    ("7x7 stride 2", "f32", 2, 3, 24, 30, 26, 7, 7, 2, 2, 3, 3),
    ("too long for LDS", "f32", 1, 3, 4, 3, 5000, 3, 3, 1, 1, 1, 1),
    ("bf16 5x5", "bf16", 8, 33, 16, 15, 17, 5, 5, 1, 1, 2, 2),
    ("bf16 stride 3", "bf16", 5, 16, 40, 19, 16, 3, 3, 3, 3, 1, 1),
    ("four pixels, sixteen channels", "f32", 40, 32, 64, 40, 52, 3, 3, 1, 1, 1, 1),
    ("stride 3 past a 1x1 filter, more channels", "f32", 4, 32, 16, 13, 11, 1, 1, 3, 3, 0, 0),
    ("7x7 stride 2, four pixels", "f32", 8, 6, 64, 112, 112, 7, 7, 2, 2, 3, 3),
    ("few channels", "f32", 16, 2, 6, 50, 50, 3, 3, 1, 1, 0, 0),
    ("towards few channels", "f32", 32, 40, 3, 32, 32, 3, 3, 1, 1, 1, 1),
]

# pixels per thread and channels per pass of the forward pass and of the data gradient, or "plain"
PLANS = {
    "four pixels per thread": ("4x16", "4x16"), "one pixel images": ("1x16", "plain"), "four channels per pass": ("1x4", "plain"),
    "stride 3 past a 1x1 filter": ("1x16", "plain"), "7x7 stride 2": ("1x4", "1x4"),
    "too long for LDS": ("plain", "plain"),
    "four pixels, sixteen channels": ("4x16", "4x16"),
    "7x7 stride 2, four pixels": ("4x4", "4x4"), "few channels": ("1x4", "plain"), "towards few channels": ("1x16", "plain"),
}
IMAGES = {"several images per workgroup": 4, "stride 3 past a 1x1 filter": 3, "one pixel images": 64, "stride 3 past a 1x1 filter, more channels": 3}


def plan_of(d, op):
    m = re.search(r"^conv_lds .*\((\d) per thread\) ch/pass=(\d+) img/tile=(\d+)", B.cac_describe_plan(d, op))
    return (f"{m[1]}x{m[2]}", int(m[3])) if m else ("plain", 1)


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_forward_and_data_gradient(case):
    import torch
    from gpu_util import Guarded, download, upload
    name, dtype, N, C, K, H, W, R, S, sh, sw, ph, pw = case
    dt = synth.F32 if dtype == "f32" else synth.BF16
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    d = B.make_desc(N, C, K, H, W, R, S, sh, sw, ph, pw, 1, 1, dtype=B.F32 if dtype == "f32" else B.BF16)
    assert B.cac_workspace_size(d, B.OP_FWD_AND_COMPRESS) == 0, "no MFMA plan: the case is here for the float kernel"
    fwd, dx = (plan_of(d, op) for op in (B.OP_FWD_AND_COMPRESS, B.OP_BWD_DATA))
    assert (fwd[0], dx[0]) == PLANS.get(name, ("1x16", "1x16"))
    assert fwd[1] == IMAGES.get(name, 1)
    P, Q = B.cac_out_shape(d)
    rng = np.random.default_rng(sum(map(ord, name)))
    make = lambda *s: synth.to_storage(rng.standard_normal(s, dtype=np.float32), dt)  # noqa: E731
    X, Wt, b, dY = make(N, C, H, W), make(K, C, R, S), make(K), make(N, K, P, Q)
    Y, Z, dX = Guarded((N, K, P, Q), td), Guarded((N, C, H, W), td), Guarded((N, C, H, W), td)
    B.conv_fwd_and_compress(d, upload(X, dt), upload(Wt, dt), upload(b, dt), Y.t, Z.t)
    B.conv_bwd_data(d, upload(Wt, dt), upload(dY, dt), dX.t)
    torch.cuda.synchronize()
    Y.check("Y"), Z.check("Z"), dX.check("dX")
    g = oracle.ConvGeom(N, C, K, H, W, R, S, sh, sw, ph, pw)
    f = [a.astype(np.float64) for a in (X, Wt, b, dY)]
    # float sums of at most 35 * 49 terms of either sign: sqrt(1715) * 2^-24 = 2.5e-6 of the result; a bfloat16 result
    # is rounded once, by at most 2^-8 of every value
    tol = 1e-5 + (0 if dtype == "f32" else 2.0 ** -8)
    for what, out, want in (("Y", Y, oracle.conv_fwd(g, f[0], f[1], f[2])), ("dX", dX, oracle.conv_dx(g, f[1], f[3]))):
        got = download(out.t)
        assert np.array_equal(got == 0, want == 0) or what == "Y", "pixels that no tap reaches are exactly zero, and only they"
        for n in range(N):
            norm = np.linalg.norm(want[n])
            assert np.linalg.norm(got[n] - want[n]) <= tol * norm, (name, what, n)


@pytest.mark.parametrize("case", [
    # name, dtype, N, C, K, H, W, R, S, stride, pad
    ("3x3", "f32", 2, 16, 18, 9, 11, 3, 3, 1, 1),
    ("3x3, four pixels per thread", "f32", 40, 32, 64, 40, 52, 3, 3, 1, 1),
    ("5x5 stride 2", "f32", 3, 5, 16, 12, 13, 5, 5, 2, 2),
    ("bf16 5x5", "bf16", 2, 9, 16, 10, 10, 5, 5, 1, 2),
], ids=lambda c: c[0])
def test_taps_outside_the_image_are_skipped(case):
    """An infinite or NaN weight makes an output non-finite only where its tap meets a pixel: padding is no pixel."""
    import torch
    from gpu_util import Guarded, download, upload
    name, dtype, N, C, K, H, W, R, S, st, pad = case
    dt, td = (synth.F32, torch.float32) if dtype == "f32" else (synth.BF16, torch.bfloat16)
    d = B.make_desc(N, C, K, H, W, R, S, st, st, pad, pad, 1, 1, dtype=B.F32 if dtype == "f32" else B.BF16, has_bias=0)
    assert all(B.cac_describe_plan(d, op).startswith("conv_lds") for op in (B.OP_FWD_AND_COMPRESS, B.OP_BWD_DATA))
    P, Q = B.cac_out_shape(d)
    rng = np.random.default_rng(5)
    make = lambda *s: synth.to_storage(rng.standard_normal(s, dtype=np.float32), dt)  # noqa: E731
    X, Wt, dY = make(N, C, H, W), make(K, C, R, S), make(N, K, P, Q)
    Wt[0, 1, 0, 0], Wt[K - 1, 0, R - 1, 1], Wt[2, C - 1, 1, S - 1] = np.inf, np.nan, -np.inf
    Y, Z, dX = Guarded((N, K, P, Q), td), Guarded((N, C, H, W), td), Guarded((N, C, H, W), td)
    B.conv_fwd_and_compress(d, upload(X, dt), upload(Wt, dt), None, Y.t, Z.t)
    B.conv_bwd_data(d, upload(Wt, dt), upload(dY, dt), dX.t)
    torch.cuda.synchronize()
    g = oracle.ConvGeom(N, C, K, H, W, R, S, st, st, pad, pad)
    f = [a.astype(np.float64) for a in (X, Wt, dY)]
    tol = 1e-5 + (0 if dtype == "f32" else 2.0 ** -8)   # as above
    for what, out, want in (("Y", Y, oracle.conv_fwd(g, f[0], f[1], np.zeros(K))), ("dX", dX, oracle.conv_dx(g, f[1], f[2]))):
        out.check(what)
        got, ok = download(out.t), np.isfinite(want)
        assert 0 < ok.sum() < ok.size
        assert np.array_equal(np.isfinite(got), ok), (name, what)
        assert np.linalg.norm(got[ok] - want[ok]) <= tol * np.linalg.norm(want[ok]), (name, what)
