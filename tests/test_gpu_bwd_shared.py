"""The combined backward call where its two launches share work -- the data gradient's repacks in the weight gradient's launch, the
slice sum in the data gradient's -- against the separate calls, bit for bit: every kernel that can carry the slices, filters that
divide nothing, the channels-last copy of both kinds, cleared pixels, and the filter laid out by the weight gradient's own waves."""
from __future__ import annotations

import pytest

from paper_2409_11902_amd import binding as B
from paper_2409_11902_amd import synth

pytestmark = pytest.mark.gpu

ROOM, SUM = "repack in its launch", "in the launch of it, the slice sum"
CASES = [
    # name, N, C, K, H, W, R, stride, what the plan says
    ("waves", 112, 80, 72, 7, 7, 3, 1, (ROOM, SUM)),
    ("waves, eight to a tile, odd channels", 10, 41, 131, 9, 10, 3, 1, (ROOM, SUM)),
    ("large wave tiles", 169, 33, 70, 14, 14, 3, 1, (ROOM, SUM)),
    ("gather in place", 16, 32, 32, 16, 16, 3, 1, (ROOM, SUM)),
    ("gather, channels-last copy by elements", 24, 45, 39, 7, 9, 3, 1, (ROOM, SUM)),
    ("gather, channels-last copy in blocks", 6, 70, 37, 6, 6, 3, 1, (ROOM,)),
    ("by waves, four classes", 19, 40, 48, 9, 11, 3, 2, (ROOM, SUM)),
    ("four parity classes", 30, 64, 32, 16, 24, 3, 2, (ROOM, SUM)),
    ("gather, four classes", 2, 40, 48, 9, 149, 3, 2, (ROOM, SUM)),
    ("pixels to clear", 30, 40, 48, 10, 11, 1, 2, (ROOM, SUM)),
    ("pointwise", 40, 40, 24, 24, 20, 1, 1, (ROOM, SUM)),
    ("pointwise by waves", 40, 40, 300, 7, 7, 1, 1, (ROOM, SUM)),
    ("filter by the waves that wait", 112, 512, 512, 7, 7, 3, 1, (ROOM,)),
    ("filter by the waves that wait, 1x1", 64, 512, 2048, 7, 7, 1, 1, (ROOM, SUM)),
    ("filter by the waves that wait, rows past the last channel", 1, 1056, 976, 4, 4, 1, 1, (ROOM,)),
    ("filter by the waves that wait, rows past the last channel, 3x3", 5, 672, 304, 12, 12, 3, 1, (ROOM,)),
    ("no room", 64, 100, 130, 28, 28, 3, 1, ("in the launch of the data gradient's repack",)),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_shared_launches_are_bit_identical_to_the_separate_calls(case):
    import torch
    from gpu_util import Guarded, upload, workspace
    name, N, C, K, H, W, R, st, words = case
    spec = synth.LayerSpec(name, N, C, K, H, W, R, R, st, R // 2)
    d = B.desc_from_spec(spec)
    plan = B.cac_describe_plan(d, B.OP_BWD_WEIGHT_AND_DATA)
    assert all(w in plan for w in words), plan
    t = synth.make_inputs(spec, "bwd-shared", tensors=("X", "W", "dY"))
    X, Wt, dY = (upload(t[n], spec.dtype) for n in ("X", "W", "dY"))
    hp, wp, _, _ = B.cac_pooled_shape(d)
    Z = torch.empty((N, C, hp, wp), dtype=torch.bfloat16, device="cuda:0")
    B.cac_compress(d, X, Z)
    out = []
    for both in (False, True, True):
        dW, dX = Guarded((K, C, R, R), torch.float32), Guarded((N, C, H, W), torch.bfloat16)
        if both:
            ws = workspace(d, B.OP_BWD_WEIGHT_AND_DATA)
            ws.fill_(0xFF)   # stale contents must not matter (all-ones floats are NaN)
            B.conv_bwd_weight_and_data(d, Z, Wt, dY, dW.t, dX.t, ws)
        else:
            B.conv_bwd_weight_compressed(d, Z, dY, dW.t, workspace(d, B.OP_BWD_WEIGHT_COMPRESSED))
            B.conv_bwd_data(d, Wt, dY, dX.t, workspace(d, B.OP_BWD_DATA))
        torch.cuda.synchronize()
        dW.check("dW"), dX.check("dX")
        out.append((dW.t.view(torch.int32), dX.t.view(torch.int16)))
    for o in out[1:]:
        assert torch.equal(out[0][0], o[0]) and torch.equal(out[0][1], o[1]), name


@pytest.mark.parametrize("k", [1, 2])
def test_data_gradient_may_take_the_place_of_the_record(k):
    """Pixels without a tap are cleared, and not while the weight gradient reads the record that lies there."""
    import torch
    from gpu_util import upload, workspace
    N, C, K, H, W = 30, 40, 48, 10, 12
    spec = synth.LayerSpec("in place", N, C, K, H, W, 1, 1, 2, 0)
    d = B.desc_from_spec(spec, pool_kh=k, pool_kw=k)
    assert ROOM in B.cac_describe_plan(d, B.OP_BWD_WEIGHT_AND_DATA)
    t = synth.make_inputs(spec, "bwd-in-place", tensors=("X", "W", "dY"))
    X, Wt, dY = (upload(t[n], spec.dtype) for n in ("X", "W", "dY"))
    hp, wp, _, _ = B.cac_pooled_shape(d)
    Z = torch.empty((N, C, hp, wp), dtype=torch.bfloat16, device="cuda:0")
    B.cac_compress(d, X, Z)
    dW, dX = torch.empty((K, C, 1, 1), dtype=torch.float32, device="cuda:0"), torch.empty_like(X)
    B.conv_bwd_weight_compressed(d, Z, dY, dW, workspace(d, B.OP_BWD_WEIGHT_COMPRESSED))
    B.conv_bwd_data(d, Wt, dY, dX, workspace(d, B.OP_BWD_DATA))
    dW2, dX2 = torch.empty_like(dW), torch.empty_like(dX)
    Z2 = dX2.view(-1)[dX2.numel() - Z.numel():]   # the record lies in the last bytes of dX
    Z2.copy_(Z.view(-1))
    B.conv_bwd_weight_and_data(d, Z2, Wt, dY, dW2, dX2, workspace(d, B.OP_BWD_WEIGHT_AND_DATA))
    torch.cuda.synchronize()
    assert torch.equal(dW.view(torch.int32), dW2.view(torch.int32)) and torch.equal(dX.view(torch.int16), dX2.view(torch.int16))
