"""Host-only: the kernels turn a flat pixel number into its row and column with a multiply-high, which is the exact
quotient only up to a pixel that depends on the row length.  No layer may be planned for such a kernel on a map that
reaches past it (the plain kernels divide)."""
from __future__ import annotations

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
