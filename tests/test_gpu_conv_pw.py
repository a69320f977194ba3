"""GPU parity of the 1 x 1 stride-1 kernel (conv_pw.hip) at the edges of what it takes: planes of every store width and
of odd size, several images per tile, tiles that end inside a plane, ragged channel counts on both sides, both
workgroup shapes, the filter read as it lies and repacked, and the pooled record formed on the way."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2409_11902_amd import binding as B
from paper_2409_11902_amd import synth

pytestmark = pytest.mark.gpu

# a result is rounded to bfloat16 once, by at most 2^-8 of its value; float sums of at most 850 terms add 1.8e-6
TOL = 2.0 ** -8 + 1e-5

CASES = [
    # name, N, C, K, H, W, k, pooled on the way
    ("rows of a multiple of 4, tiles of whole row pairs", 3, 96, 40, 20, 28, 2, True),
    ("tile of one row pair", 2, 64, 64, 6, 100, 2, True),
    ("longest rows that are pooled on the way", 1, 32, 16, 4, 128, 2, True),
    ("longer rows", 1, 32, 16, 4, 132, 2, False),
    ("128 output channels, filter as it lies", 128, 64, 130, 16, 32, 2, True),
    ("128 output channels, filter repacked", 300, 200, 256, 14, 16, 2, True),
    ("odd height, rows of a multiple of 4", 4, 48, 65, 15, 12, 2, False),
    ("8-byte stores", 3, 33, 70, 14, 14, 2, False),
    ("4-byte stores", 5, 72, 100, 13, 10, 2, False),
    ("odd planes, several images per tile", 37, 130, 64, 7, 7, 2, False),
    ("odd planes longer than a tile", 4, 100, 96, 17, 19, 1, False),
    ("small even planes, batch not a multiple", 53, 16, 24, 4, 4, 1, False),
    ("one pixel", 70, 400, 33, 1, 1, 1, False),
    ("tile 4", 3, 64, 32, 16, 16, 4, False),
]


# layers that the planner leaves to the gather kernel: channels of a tile shared out, and one workgroup for all of them
GATHER = [
    ("long sum, few workgroups", 2, 512, 64, 7, 8, 2, False),
    ("long sum, odd planes", 3, 530, 70, 5, 5, 4, False),
    ("planes of four pixels", 270, 260, 850, 2, 2, 1, False),
    ("the record out of the repack", 40, 45, 20, 8, 8, 2, False),
]


@pytest.mark.parametrize("case", CASES + GATHER, ids=[c[0] for c in CASES + GATHER])
def test_forward_record_and_data_gradient(case):
    import torch
    from gpu_util import Guarded, download, upload, workspace
    name, N, C, K, H, W, k, pooled = case
    spec = synth.LayerSpec(name, N, C, K, H, W, 1, 1, 1, 0, k)
    t = synth.make_inputs(spec, "conv-pw")
    d = B.desc_from_spec(spec)
    plan = B.cac_describe_plan(d, B.OP_FWD_AND_COMPRESS)
    assert plan.startswith("gather" if case in GATHER else "pointwise") and ("pooled on the way" in plan) == pooled, plan
    X, Wt, b, dY = (upload(t[n], spec.dtype) for n in ("X", "W", "b", "dY"))
    hp, wp, _, _ = B.cac_pooled_shape(d)
    Y, dX = Guarded((N, K, H, W), torch.bfloat16), Guarded((N, C, H, W), torch.bfloat16)
    Z, Z1 = Guarded((N, C, hp, wp), torch.bfloat16), Guarded((N, C, hp, wp), torch.bfloat16)
    B.conv_fwd_and_compress(d, X, Wt, b, Y.t, Z.t, workspace(d, B.OP_FWD_AND_COMPRESS))
    B.cac_compress(d, X, Z1.t)
    B.conv_bwd_data(d, Wt, dY, dX.t, workspace(d, B.OP_BWD_DATA))
    torch.cuda.synchronize()
    for buf, what in ((Y, "Y"), (Z, "Z"), (Z1, "Z"), (dX, "dX")):
        buf.check(what)
    assert torch.equal(Z.t.view(torch.int16), Z1.t.view(torch.int16)), "the record is bit for bit the stand-alone kernel's"
    g = oracle.ConvGeom(N, C, K, H, W, 1, 1, 1, 1, 0, 0)
    f = {n: t[n].astype(np.float64) for n in ("X", "W", "b", "dY")}
    for what, out, want in (("Y", Y, oracle.conv_fwd(g, f["X"], f["W"], f["b"])), ("dX", dX, oracle.conv_dx(g, f["W"], f["dY"]))):
        got = download(out.t)
        for n in range(N):
            assert np.linalg.norm(got[n] - want[n]) <= TOL * np.linalg.norm(want[n]), (name, what, n)
