"""Nine-tap launches by waves (csrc/conv_wave.hip) against the oracle, at the edges of its tiles: maps that share a tile of 64
pixels, a last tile that is not full, stages that are not full, rows of odd length, one and two items to a lane, four and eight
waves to a tile, filters other than 3 x 3 with padding 1."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2409_11902_amd import binding as B
from paper_2409_11902_amd import synth

pytestmark = pytest.mark.gpu

# One rounding to bfloat16 moves a value by at most 2^-8 of it, and an image's rel-L2 by no more; the float sums (at most
# 9 * 1000 terms of products exact in float) add about sqrt(9000) * 2^-24 = 6e-6.
TOL = 2.0 ** -8 + 1e-5

CASES = [
    # name, N, C, K, H, W, R, S, pad_h, pad_w, stride, by waves: forward, data gradient
    ("whole images of 16 pixels", 68, 200, 130, 4, 4, 3, 3, 1, 1, 1, True, True),
    ("five tiles and a bit of 25", 53, 64, 100, 5, 5, 3, 3, 1, 1, 1, True, True),
    ("rows of 7", 20, 80, 72, 7, 7, 3, 3, 1, 1, 1, True, True),
    ("rows of 14", 12, 130, 96, 14, 14, 3, 3, 1, 1, 1, True, True),
    ("last stage partial, 4-byte stores", 11, 69, 75, 9, 14, 3, 3, 1, 1, 1, True, True),
    ("rows of one item and a bit", 9, 96, 64, 10, 9, 3, 3, 1, 1, 1, True, True),
    ("two items to a lane, odd rows", 3, 300, 64, 9, 55, 3, 3, 1, 1, 1, True, True),
    ("eight waves, one tile", 1, 1000, 16, 5, 5, 3, 3, 1, 1, 1, True, False),
    ("eight waves, 32 channels", 2, 24, 700, 9, 9, 3, 3, 1, 1, 1, True, True),
    ("stride 2", 16, 72, 160, 28, 28, 3, 3, 1, 1, 2, True, True),
    ("stride 2, odd extents", 17, 90, 193, 15, 27, 3, 3, 1, 1, 2, True, True),
    ("stride 2, maps of 4 pixels", 8, 464, 64, 4, 5, 3, 3, 1, 1, 2, True, True),
    ("stride 2, one pixel", 5, 40, 70, 1, 1, 3, 3, 1, 1, 2, False, True),
    ("stride 2, last stage partial, M tail", 9, 69, 300, 14, 14, 3, 3, 1, 1, 2, True, True),
    ("stride 2, odd rows of dY, even of dX", 33, 24, 97, 11, 18, 3, 3, 1, 1, 2, True, True),
    ("stride 2, even rows of dY, odd of dX", 3, 33, 1000, 12, 15, 3, 3, 1, 1, 2, True, True),
    ("no padding", 12, 80, 72, 9, 10, 3, 3, 0, 0, 1, True, True),
    ("padding 2", 12, 80, 72, 9, 10, 3, 3, 2, 2, 1, True, True),
    ("padding 3 and 1", 12, 81, 72, 8, 11, 3, 3, 3, 1, 1, True, True),
    ("1x9 padding 4", 12, 80, 72, 8, 13, 1, 9, 0, 4, 1, True, True),
    ("9x1 padding 4", 12, 80, 72, 13, 8, 9, 1, 4, 0, 1, True, True),
    # rows of padding alone below an image, and a tile that starts in them
    ("maps of 16 pixels, padding 4", 8, 128, 128, 4, 4, 3, 3, 4, 4, 1, True, False),
    ("rows of 7, padding 5", 4, 256, 64, 7, 7, 3, 3, 5, 5, 1, True, False),
    ("rows of 14, padding 4", 16, 64, 64, 14, 14, 3, 3, 4, 4, 1, True, True),
    ("padding 5 and 1", 12, 80, 72, 9, 10, 3, 3, 5, 1, 1, True, True),
    ("1x9 padding 2 and 4", 12, 80, 72, 8, 13, 1, 9, 2, 4, 1, True, True),
    ("9x1 padding 12", 8, 100, 90, 3, 5, 9, 1, 12, 0, 1, True, False),
    ("1x9 stride 2", 12, 80, 72, 20, 28, 1, 9, 0, 4, 2, True, False),
    ("1x9 stride 2, tall maps", 8, 256, 256, 40, 20, 1, 9, 0, 4, 2, True, False),
    ("1x9 stride 2, padding 3 and 4", 12, 80, 72, 20, 28, 1, 9, 3, 4, 2, True, False),
    ("stride 2, padding 6 and 5", 12, 80, 72, 5, 6, 3, 3, 6, 5, 2, True, False),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_forward_and_data_gradient(case):
    import torch
    from gpu_util import Guarded, download, upload, workspace
    name, N, C, K, H, W, R, S, ph, pw, st, fwd, dx = case
    d = B.make_desc(N, C, K, H, W, R, S, st, st, ph, pw)
    for op, waves in ((B.OP_FWD_AND_COMPRESS, fwd), (B.OP_BWD_DATA, dx)):
        plan = B.cac_describe_plan(d, op)
        assert ("by waves" in plan) == waves, plan
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
    for out, want in ((Y, oracle.conv_fwd(g, f[0], f[1], f[2])), (dX, oracle.conv_dx(g, f[1], f[3]))):
        got = download(out.t)
        for n in range(N):
            err = np.linalg.norm(got[n] - want[n]) / np.linalg.norm(want[n])
            assert err <= TOL, (name, n, err)


# Layers beside the line that keep the stages shared (csrc/conv_dx2.hip): 16-byte and dword stores, a tile ending inside a block.
SHARED = [("16-byte stores", 30, 64, 32, 16, 24), ("tile ends inside a block", 24, 130, 40, 30, 28), ("odd number of dY elements", 135, 33, 31, 13, 14)]


@pytest.mark.parametrize("case", SHARED, ids=[c[0] for c in SHARED])
def test_stride_2_data_gradient_with_shared_stages(case):
    import torch
    from gpu_util import Guarded, download, upload, workspace
    name, N, C, K, H, W = case
    d = B.make_desc(N, C, K, H, W, 3, 3, 2, 2, 1, 1)
    plan = B.cac_describe_plan(d, B.OP_BWD_DATA)
    assert "four parity classes" in plan and "by waves" not in plan, plan
    P, Q = B.cac_out_shape(d)
    rng = np.random.default_rng(N)
    Wt, dY = (synth.to_storage(rng.standard_normal(s, dtype=np.float32), synth.BF16) for s in ((K, C, 3, 3), (N, K, P, Q)))
    dX = Guarded((N, C, H, W), torch.bfloat16)
    B.conv_bwd_data(d, upload(Wt, synth.BF16), upload(dY, synth.BF16), dX.t, workspace(d, B.OP_BWD_DATA))
    torch.cuda.synchronize()
    dX.check("dX")
    want = oracle.conv_dx(oracle.ConvGeom(N, C, K, H, W, 3, 3, 2, 2, 1, 1), Wt.astype(np.float64), dY.astype(np.float64))
    got = download(dX.t)
    for n in range(N):
        assert np.linalg.norm(got[n] - want[n]) <= TOL * np.linalg.norm(want[n]), (name, n)
