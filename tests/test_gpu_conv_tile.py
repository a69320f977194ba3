"""GPU parity of the nine-tap kernel with large wave tiles (conv_tile.hip) and of the stride-2 data gradient that
computes all parity classes in one launch (conv_dx2.hip) at the edges of what they take: rows of
odd length and of every store width, tiles that end inside a block, several images per tile and a batch they do not
divide, ragged channel counts on both sides, stride 2, items that fill a thread once and twice."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2409_11902_amd import binding as B
from paper_2409_11902_amd import synth

pytestmark = pytest.mark.gpu

# bfloat16 keeps 8 significant bits: rounding to nearest moves a value by at most half a unit in the last place, 2^-8
# of it, and an image's rel-L2 by no more (1.65e-3 in the mean over mantissas, 1.98e-3 seen on an image of 1600
# values); the float sums (at most 9 * 136 terms of products exact in float) add about sqrt(1224) * 2^-24 = 2e-6
TOL = 2.0 ** -8 + 1e-5

CASES = [
    # name, N, C, K, H, W, stride
    ("16-byte stores, one block short", 80, 32, 64, 20, 28, 1),
    ("8-byte stores, rows of 14", 165, 64, 128, 14, 14, 1),
    ("4-byte stores", 80, 40, 72, 9, 22, 1),
    ("2-byte stores, rows of 7", 330, 32, 136, 7, 7, 1),
    ("odd rows longer than an item", 80, 24, 80, 12, 9, 1),
    ("odd rows, odd planes", 40, 35, 65, 11, 27, 1),
    ("batch not a multiple of the images per tile", 1201, 16, 64, 5, 6, 1),
    ("wide rows, two items per thread", 24, 33, 64, 30, 56, 1),
    ("whole blocks only", 165, 32, 64, 16, 16, 1),
    ("stride 2", 160, 32, 80, 28, 28, 2),
    ("stride 2, odd extents", 160, 20, 130, 27, 15, 2),
    ("channels past one block of 32", 80, 65, 33, 18, 20, 1),
    ("256 output channels", 160, 40, 256, 10, 14, 1),
    ("stages of 16 channels, last one partial", 90, 37, 64, 31, 52, 1),
    ("stages of 16 channels, odd rows", 170, 48, 60, 22, 41, 1),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_forward_and_data_gradient(case):
    import torch
    from gpu_util import Guarded, download, upload, workspace
    name, N, C, K, H, W, st = case
    spec = synth.LayerSpec(name, N, C, K, H, W, stride=st)
    t = synth.make_inputs(spec, "conv-tile")
    d = B.desc_from_spec(spec)
    assert B.cac_describe_plan(d, B.OP_FWD_AND_COMPRESS).startswith("tile="), "the case is here for that kernel"
    X, Wt, b, dY = (upload(t[n], spec.dtype) for n in ("X", "W", "b", "dY"))
    hp, wp, _, _ = B.cac_pooled_shape(d)
    Y, Z = Guarded((N, K, spec.P, spec.Q), torch.bfloat16), Guarded((N, C, hp, wp), torch.bfloat16)
    dX = Guarded((N, C, H, W), torch.bfloat16)
    B.conv_fwd_and_compress(d, X, Wt, b, Y.t, Z.t, workspace(d, B.OP_FWD_AND_COMPRESS))
    B.conv_bwd_data(d, Wt, dY, dX.t, workspace(d, B.OP_BWD_DATA))
    torch.cuda.synchronize()
    Y.check("Y"), Z.check("Z"), dX.check("dX")
    g = oracle.ConvGeom(N, C, K, H, W, 3, 3, st, st, 1, 1)
    f = {n: t[n].astype(np.float64) for n in ("X", "W", "b", "dY")}
    for out, want in ((Y, oracle.conv_fwd(g, f["X"], f["W"], f["b"])), (dX, oracle.conv_dx(g, f["W"], f["dY"]))):
        got = download(out.t)
        # every image by itself: an error in the last one must not hide behind the others
        for n in range(N):
            err = np.linalg.norm(got[n] - want[n]) / np.linalg.norm(want[n])
            assert err <= TOL, (name, n, err)


GENERAL = [
    # name, N, C, K, H, W, R, S, pad_h, pad_w, stride: what else the planner sends there -- other paddings, one-row and
    # one-column filters, and tensors whose last load or store ends in the middle of a dword
    ("3x3 without padding", 90, 32, 64, 20, 28, 3, 3, 0, 0, 1),
    ("3x3 without padding, stride 2", 170, 24, 72, 29, 30, 3, 3, 0, 0, 2),
    ("3x3 padding 2", 80, 40, 48, 18, 20, 3, 3, 2, 2, 1),
    ("3x3 padding 3 and 1", 80, 17, 64, 15, 24, 3, 3, 3, 1, 1),
    ("1x9", 90, 32, 64, 20, 28, 1, 9, 0, 0, 1),
    ("1x9 padding 4", 90, 33, 70, 14, 21, 1, 9, 0, 4, 1),
    ("9x1", 90, 32, 64, 28, 20, 9, 1, 0, 0, 1),
    ("9x1 padding 4", 90, 40, 65, 22, 15, 9, 1, 4, 0, 1),
    ("odd numbers of elements", 101, 35, 65, 11, 27, 3, 3, 1, 1, 1),
    ("odd numbers of elements, rows of 7", 481, 33, 67, 7, 7, 3, 3, 1, 1, 1),
]


@pytest.mark.parametrize("case", GENERAL, ids=[c[0] for c in GENERAL])
def test_other_nine_tap_filters(case):
    import torch
    from gpu_util import Guarded, download, upload, workspace
    name, N, C, K, H, W, R, S, ph, pw, st = case
    d = B.make_desc(N, C, K, H, W, R, S, st, st, ph, pw)
    fwd, dx = (B.cac_describe_plan(d, op).replace("class(0,0): ", "") for op in (B.OP_FWD_AND_COMPRESS, B.OP_BWD_DATA))
    assert fwd.startswith("tile=") and (st == 2 or dx.startswith("tile=")), (fwd, dx)
    P, Q = B.cac_out_shape(d)
    rng = np.random.default_rng(sum(map(ord, name)))
    make = lambda *s: synth.to_storage(rng.standard_normal(s, dtype=np.float32), synth.BF16)  # noqa: E731
    X, Wt, b, dY = make(N, C, H, W), make(K, C, R, S), make(K), make(N, K, P, Q)
    hp, wp, _, _ = B.cac_pooled_shape(d)
    Y, Z, dX = (Guarded(s, torch.bfloat16) for s in ((N, K, P, Q), (N, C, hp, wp), (N, C, H, W)))
    up = lambda a: upload(a, synth.BF16)  # noqa: E731
    B.conv_fwd_and_compress(d, up(X), up(Wt), up(b), Y.t, Z.t, workspace(d, B.OP_FWD_AND_COMPRESS))
    B.conv_bwd_data(d, up(Wt), up(dY), dX.t, workspace(d, B.OP_BWD_DATA))
    torch.cuda.synchronize()
    Y.check("Y"), Z.check("Z"), dX.check("dX")
    g = oracle.ConvGeom(N, C, K, H, W, R, S, st, st, ph, pw)
    f = [a.astype(np.float64) for a in (X, Wt, b, dY)]
    for what, out, want in (("Y", Y, oracle.conv_fwd(g, f[0], f[1], f[2])), ("dX", dX, oracle.conv_dx(g, f[1], f[3]))):
        got = download(out.t)
        for n in range(N):
            assert np.linalg.norm(got[n] - want[n]) <= TOL * np.linalg.norm(want[n]), (name, what, n)


STRIDE2 = [
    # name, N, C, K, H, W: dY rows of a multiple of 4, of 2, of odd length; a last input row that only some classes have
    ("16-byte stores", 3, 64, 96, 16, 24),
    ("8-byte stores, odd height", 5, 40, 33, 13, 20),
    ("4-byte stores, rows of 7", 9, 72, 64, 14, 14),
    ("odd rows, odd height", 4, 33, 65, 11, 18),
    ("several images per tile, batch not a multiple", 23, 32, 40, 7, 8),
    ("one row of pixels", 6, 16, 16, 1, 6),
    ("one column of pairs", 6, 20, 16, 9, 2),
    ("tile ends inside a block", 2, 130, 70, 30, 28),
    ("long rows", 1, 16, 48, 6, 120),
    ("odd number of dY elements", 5, 33, 65, 13, 14),
]


@pytest.mark.parametrize("case", STRIDE2, ids=[c[0] for c in STRIDE2])
def test_stride_2_data_gradient(case):
    import torch
    from gpu_util import Guarded, download, upload, workspace
    name, N, C, K, H, W = case
    spec = synth.LayerSpec(name, N, C, K, H, W, stride=2)
    t = synth.make_inputs(spec, "conv-dx2", tensors=("W", "dY"))
    d = B.desc_from_spec(spec)
    assert "four parity classes" in B.cac_describe_plan(d, B.OP_BWD_DATA), "the case is here for that kernel"
    Wt, dY = upload(t["W"], spec.dtype), upload(t["dY"], spec.dtype)
    dX = Guarded((N, C, H, W), torch.bfloat16)
    B.conv_bwd_data(d, Wt, dY, dX.t, workspace(d, B.OP_BWD_DATA))
    torch.cuda.synchronize()
    dX.check("dX")
    want = oracle.conv_dx(oracle.ConvGeom(N, C, K, H, W, 3, 3, 2, 2, 1, 1), t["W"].astype(np.float64), t["dY"].astype(np.float64))
    got = download(dX.t)
    for n in range(N):
        for a0 in range(min(2, H)):
            for b0 in range(2):     # every class of every image by itself
                w = want[n, :, a0::2, b0::2]
                assert np.linalg.norm(got[n, :, a0::2, b0::2] - w) <= TOL * np.linalg.norm(w), (name, n, a0, b0)
