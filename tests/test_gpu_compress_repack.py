"""GPU parity of forward passes whose pooling launch carries the filter's repack: every form of the pooling kernel (rows of 10,
12 and 14, rows below 8 and above, tiles of 1 to 4, ragged ones), filters of whole and of ragged blocks, a record of a single
block; and of passes on channels-last copies, which pool by themselves.  The plan says which."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2409_11902_amd import binding as B
from paper_2409_11902_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    # N, C, K, H, W, kh, kw, R, stride, shared launch
    (48, 33, 65, 10, 10, 2, 2, 3, 1, True),
    (40, 64, 130, 12, 12, 2, 2, 3, 1, True),
    (40, 72, 96, 14, 14, 2, 2, 3, 1, True),
    (400, 24, 16, 15, 14, 2, 2, 3, 1, True),   # rows of 14, an odd number of them: chunks
    (3, 20, 24, 15, 14, 2, 2, 3, 1, False),
    (90, 48, 64, 7, 7, 2, 2, 3, 1, False),
    (150, 16, 64, 6, 5, 4, 4, 3, 1, False),
    (20, 40, 70, 27, 30, 4, 4, 3, 1, True),
    (20, 40, 70, 27, 30, 1, 1, 3, 1, True),
    (20, 40, 70, 27, 30, 2, 4, 3, 1, True),
    (20, 40, 70, 27, 30, 4, 2, 3, 1, True),
    (24, 40, 70, 28, 28, 1, 1, 3, 2, True),
    (2, 300, 64, 13, 13, 2, 2, 1, 1, True),
    # rows below 8: chunks of 4
    (200, 16, 8, 6, 6, 1, 1, 3, 1, True),
    (200, 16, 8, 6, 6, 2, 2, 3, 1, True),
    (200, 16, 8, 6, 6, 4, 4, 3, 1, True),
    (200, 16, 8, 6, 6, 2, 4, 3, 1, True),
    (200, 40, 70, 5, 7, 4, 2, 1, 1, True),
    (40, 200, 64, 3, 3, 2, 2, 1, 1, True),
    (16, 8, 8, 10, 6, 4, 4, 3, 1, True),
    (1, 8, 8, 3, 3, 2, 2, 1, 1, True),         # one block of each
    (1, 8, 8, 3, 3, 2, 2, 3, 1, False),
]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_forward_and_record(case):
    import torch
    from gpu_util import Guarded, download, upload, workspace
    N, C, K, H, W, kh, kw, R, stride, shared = case
    spec = synth.LayerSpec("compress-repack-%d-%d-%d-%d-%d" % case[:5], N, C, K, H, W, R, R, stride, R // 2)
    t = synth.make_inputs(spec, "compress-repack", tensors=("X", "W", "b"))
    d = B.desc_from_spec(spec, pool_kh=kh, pool_kw=kw)
    plan = B.cac_describe_plan(d, B.OP_FWD_AND_COMPRESS)
    assert ("the record in the filter's launch" in plan) == shared, plan
    X, Wt, b = (upload(t[n], spec.dtype) for n in ("X", "W", "b"))
    hp, wp, _, _ = B.cac_pooled_shape(d)
    Y, Z, Z1 = (Guarded(s, torch.bfloat16) for s in ((N, K, spec.P, spec.Q), (N, C, hp, wp), (N, C, hp, wp)))
    B.conv_fwd_and_compress(d, X, Wt, b, Y.t, Z.t, workspace(d, B.OP_FWD_AND_COMPRESS))
    B.cac_compress(d, X, Z1.t)
    torch.cuda.synchronize()
    for buf, what in ((Y, "Y"), (Z, "Z"), (Z1, "Z")):
        buf.check(what)
    assert torch.equal(Z.t.view(torch.int16), Z1.t.view(torch.int16)), "the record is bit for bit the stand-alone kernel's"
    g = oracle.ConvGeom(N, C, K, H, W, R, R, stride, stride, R // 2, R // 2)
    want = oracle.conv_fwd(g, *(t[n].astype(np.float64) for n in ("X", "W", "b")))
    # one rounding to bfloat16, at most 2^-8 of a value; float sums of at most 648 terms add 1.5e-6
    assert np.linalg.norm(download(Y.t) - want) <= (2.0 ** -8 + 1e-5) * np.linalg.norm(want)
