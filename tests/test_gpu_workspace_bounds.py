"""Every route of the forward pass and the data gradient in a workspace of exactly the size asked for, canaries on both
sides: nothing is written past it, and the results are those of a call with room to spare."""
from __future__ import annotations

import pytest

from paper_2409_11902_amd import binding as B
from paper_2409_11902_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    # name, N, C, K, H, W, R, stride, k, what the forward and the data-gradient plan have to contain
    ("large wave tiles", 80, 40, 72, 18, 20, 3, 1, 2, "tile=", "tile="),
    ("large wave tiles, Z from the repack launch", 160, 40, 72, 16, 16, 3, 1, 2, "tile=", "tile="),
    ("four classes", 9, 72, 64, 14, 14, 3, 2, 1, "gather", "four parity classes"),
    ("pointwise, filter as it lies", 2, 64, 64, 20, 20, 1, 1, 2, "pointwise", "pointwise"),
    ("pointwise, filter repacked", 3, 72, 40, 20, 20, 1, 1, 4, "pointwise", "pointwise"),
    ("gather in place", 16, 32, 32, 16, 16, 3, 1, 4, "X read in place", "dY read in place"),
    ("gather in place, Z from the repack launch", 16, 32, 32, 16, 16, 3, 1, 2, "X read in place", "dY read in place"),
    ("gather, channels-last copy", 2, 70, 33, 7, 7, 3, 1, 2, "gather", "gather"),
    ("gather, shared-out channels", 4, 256, 128, 4, 4, 3, 1, 2, "gather", "gather"),
    ("decimated copy", 3, 48, 72, 16, 24, 1, 2, 2, "keeps one pixel", "gather"),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_exact_workspace(case):
    import torch
    from gpu_util import Guarded, upload
    name, N, C, K, H, W, R, st, k, fwd, dx = case
    spec = synth.LayerSpec(name, N, C, K, H, W, R, R, st, R // 2, k)
    t = synth.make_inputs(spec, "ws")
    d = B.desc_from_spec(spec)
    assert fwd in B.cac_describe_plan(d, B.OP_FWD_AND_COMPRESS) and dx in B.cac_describe_plan(d, B.OP_BWD_DATA)
    X, Wt, b, dY = (upload(t[n], spec.dtype) for n in ("X", "W", "b", "dY"))
    hp, wp, _, _ = B.cac_pooled_shape(d)
    bf = torch.bfloat16
    runs = []
    for extra in (0, 1 << 20):
        o = dict(Y=Guarded((N, K, spec.P, spec.Q), bf), Z=Guarded((N, C, hp, wp), bf), dX=Guarded((N, C, H, W), bf),
                 dX2=Guarded((N, C, H, W), bf), dW=Guarded((K, C, R, R), torch.float32))

        def scratch(op):
            ws = Guarded((B.cac_workspace_size(d, op) + extra,), torch.uint8)
            o[f"workspace of op {op}"] = ws
            return ws.t if ws.nbytes else None
        B.conv_fwd_and_compress(d, X, Wt, b, o["Y"].t, o["Z"].t, scratch(B.OP_FWD_AND_COMPRESS))
        B.conv_bwd_data(d, Wt, dY, o["dX"].t, scratch(B.OP_BWD_DATA))
        B.conv_bwd_weight_and_data(d, o["Z"].t, Wt, dY, o["dW"].t, o["dX2"].t, scratch(B.OP_BWD_WEIGHT_AND_DATA))
        torch.cuda.synchronize()
        for n, g in o.items():
            g.check(f"{name}: {n}")
        runs.append(o)
    for n in ("Y", "Z", "dX", "dX2", "dW"):
        a, c = (r[n].t.view(torch.uint8 if n == "dW" else torch.int16) for r in runs)
        assert torch.equal(a, c), (name, n)
