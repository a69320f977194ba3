"""Host-only: the kernels turn a flat pixel number into its row and column with a multiply-high, which is the exact
quotient only up to a pixel that depends on the row length.  No layer may be planned for such a kernel on a map that
reaches past it (the plain kernels divide)."""
from __future__ import annotations

import re

import pytest

from paper_2409_11902_amd import binding as B

LIMIT = 1 << 30     # padded elements of a tensor that the matrix-core kernels take


def last_row_is_exact(rows: int, cols: int) -> bool:
    """The quotient of the map's last pixel; the error grows with the pixel, so every other one is exact with it."""
    magic = -(-(1 << 32) // cols)
    x = rows * cols - 1
    return cols == 1 or (x * magic) >> 32 == rows - 1


def multiplies(plan: str) -> bool:
    """Whether the plan's kernels divide pixels that way (the pointwise kernel does not)."""
    return "tile=" in plan and "pointwise" not in plan


@pytest.mark.parametrize("op,stride", [(B.OP_FWD_AND_COMPRESS, 1), (B.OP_FWD_AND_COMPRESS, 2), (B.OP_BWD_DATA, 1), (B.OP_BWD_DATA, 2)])
def test_no_plan_divides_inexactly(op, stride):
    planned = refused = 0
    for W in range(2, 1300):
        H = min(1 << 24, (LIMIT - 1) // (16 * W))
        d = B.make_desc(1, 16, 16, H, W, 3, 3, stride, stride, 1, 1)
        rows, cols = ((H + stride - 1) // stride, (W + stride - 1) // stride)   # of the output, or of a parity class
        if multiplies(B.cac_describe_plan(d, op)):
            planned += 1
            assert last_row_is_exact(rows, cols), (W, H)
        elif not last_row_is_exact(rows, cols):
            refused += 1
    assert planned and refused, "both sides of the rule are met"


def test_the_rule_refuses_nothing_else():
    """3 x 3 on rows of 190: pixel 23342259 (row 122853, column 189) is the first wrong one."""
    def plan(H):
        return B.cac_describe_plan(B.make_desc(1, 16, 16, H, 190, 3, 3, 1, 1, 1, 1), B.OP_FWD_AND_COMPRESS)
    assert last_row_is_exact(122853, 190) and not last_row_is_exact(122854, 190)
    assert multiplies(plan(122853)) and not multiplies(plan(122854))
    # a power of two divides exactly everywhere
    assert multiplies(B.cac_describe_plan(B.make_desc(1, 16, 16, 500000, 128, 3, 3, 1, 1, 1, 1), B.OP_FWD_AND_COMPRESS))


def rows_are_exact(units: int, blocks: int) -> bool:
    magic = -(-(1 << 32) // blocks)
    return blocks == 1 or ((units - 1) * magic) >> 32 == (units - 1) // blocks


@pytest.mark.parametrize("kernel,over", [("dw_mfma", {}), ("dw_rk", dict(dw_algo=B.DW_REDUCED_K)), ("dw_tiled", dict(dtype=B.F32))])
def test_no_weight_gradient_plan_divides_inexactly(kernel, over):
    """A weight gradient's units are numbered image by image, row block by row block; the kernels divide the number by
    an image's row blocks."""
    per_unit = {"dw_mfma": r"chunk=(\d+)img x (\d+)rows", "dw_rk": r"unit=(\d+)img x (\d+)pooled rows", "dw_tiled": r"unit=()(\d+) rows"}
    planned = refused = 0
    for i in range(0, 400, 10):
        N, H = 1 + i % 3, 500002 + 2503 * 2 * i
        plan = B.cac_describe_plan(B.make_desc(N, 128, 16, H, 2, 3, 3, 1, 1, 1, 1, **over), B.OP_BWD_WEIGHT_COMPRESSED)
        if not plan.startswith(kernel):
            refused += 1
            continue
        planned += 1
        imgs, rows = (int(x or 1) for x in re.search(per_unit[kernel], plan).groups())
        blocks = -(-(H // 2 if kernel == "dw_rk" else H) // rows)
        units = int(re.search(r"(?:units|chunks)=(\d+)", plan).group(1))
        assert units == -(-N // imgs) * blocks
        assert rows_are_exact(units, blocks), (N, H)
    assert planned
    assert refused or kernel == "dw_mfma"     # (that planner has chunks of other lengths to take)


def test_tiled_weight_gradient_divides_pooling_tiles_exactly():
    """... and a pixel's row and column by the pooling tile's extents."""
    for kh in range(1500, 1540):
        d = B.make_desc(1, 1, 1, 1 << 24, 8, 1, 1, pool_kh=kh, dtype=B.F32)
        magic = -(-(1 << 32) // kh)
        exact = all((h * magic) >> 32 == h // kh for h in range((1 << 24) - kh, 1 << 24))
        assert exact or not B.cac_describe_plan(d, B.OP_BWD_WEIGHT_COMPRESSED).startswith("dw_tiled"), kh
