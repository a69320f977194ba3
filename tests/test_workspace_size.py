"""Host-only: the scratch a call asks for is what its launches use.  Where the input is read in place there is no
channels-last copy, so the repacked filter and the float sums of shared-out channels are all that is left."""
from __future__ import annotations

import random
import re

import pytest

from paper_2409_11902_amd import binding as B

MiB = 1 << 20


def up(x, m):
    return -(-x // m) * m


def bound(d, op, plan):
    """Filter rows and columns padded to at most 64, and one plane set of floats per share of the channels."""
    n = up(2 * d.R * d.S * up(d.C_in, 64) * up(d.C_out, 64), 256)
    grid = re.search(r"grid=\d+x\d+x(\d+)", plan)
    if grid and int(grid.group(1)) > 1:
        p, q = B.cac_out_shape(d)
        n += int(grid.group(1)) * 4 * d.N * (d.C_out * p * q if op == B.OP_FWD_AND_COMPRESS else d.C_in * d.H * d.W)
    return n


def test_no_copy_area_where_the_input_is_read_in_place():
    r, seen = random.Random(3), {}
    for _ in range(6000):
        R = r.choice([1, 3, 3])
        st = r.choice([1, 1, 2])
        H = r.randint(4, 60)
        d = B.make_desc(r.randint(1, 128), r.randint(1, 600), r.randint(1, 600), H, r.choice([H, r.randint(4, 60)]), R, R, st, st, R // 2, R // 2)
        for op in (B.OP_FWD_AND_COMPRESS, B.OP_BWD_DATA):
            plan = B.cac_describe_plan(d, op)
            if "read in place" not in plan:
                continue
            kind = (op, plan.split(": ")[-1 if op == B.OP_BWD_DATA else 0].split()[0].split("=")[0])
            seen[kind] = seen.get(kind, 0) + 1
            assert B.cac_workspace_size(d, op) <= bound(d, op, plan), (d.N, d.C_in, d.C_out, d.H, d.W, R, st, plan)
    assert set(seen) == {(op, k) for op in (B.OP_FWD_AND_COMPRESS, B.OP_BWD_DATA) for k in ("tile", "pointwise", "gather")}
    assert min(seen.values()) > 50


@pytest.mark.parametrize("shape,op,limit", [
    # a record of a quarter of X must not be paid for with a scratch copy of X
    ((256, 512, 512, 14, 14, 3), B.OP_FWD_AND_COMPRESS, 9 * 512 * 512 * 2),
    ((256, 512, 512, 14, 14, 3), B.OP_BWD_DATA, 9 * 512 * 512 * 2),
    ((64, 256, 64, 56, 56, 1), B.OP_FWD_AND_COMPRESS, 256 * 64 * 2),
    ((64, 64, 16, 500, 500, 1), B.OP_FWD_AND_COMPRESS, 64 * 64 * 2),
    ((64, 256, 100, 224, 224, 3), B.OP_BWD_DATA, 9 * 256 * 128 * 2),
    # the filter read where it lies too: nothing at all
    ((2, 256, 64, 56, 56, 1), B.OP_FWD_AND_COMPRESS, 0),
])
def test_known_layers(shape, op, limit):
    N, C, K, H, W, R = shape
    d = B.make_desc(N, C, K, H, W, R, R, 1, 1, R // 2, R // 2)
    assert B.cac_workspace_size(d, op) <= up(limit, 256)


def test_decimated_copy_is_a_quarter():
    """1 x 1 stride 2 with 2 x 2 tiles: the channels-last copy keeps one pixel of four."""
    d = B.make_desc(64, 256, 512, 56, 56, 1, 1, 2, 2)
    assert "one pixel of every 2 x 2 tile" in B.cac_describe_plan(d, B.OP_FWD_AND_COMPRESS)
    assert B.cac_workspace_size(d, B.OP_FWD_AND_COMPRESS) == 2 * 64 * 28 * 28 * 256 + 2 * 256 * 512
