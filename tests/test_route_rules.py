"""Host-only: which kernel a layer is planned for, on both sides of rules whose lines were drawn from measurements."""
from __future__ import annotations

import pytest

from paper_2409_11902_amd import binding as B


@pytest.mark.parametrize("shape,k,plan,pooled", [
    # N, C, K, H, W.  The 2 x 2 record comes out of the gather's repack for nothing on rows of 4 or a multiple of 8 ...
    ((168, 45, 20, 8, 8), 2, "gather", False),
    ((168, 45, 20, 8, 8), 4, "pointwise", False),
    ((1050, 45, 20, 8, 8), 2, "pointwise", False),      # ... which no longer decides from 256 workgroups on
    ((168, 45, 20, 9, 9), 2, "pointwise", False),
    ((30, 160, 48, 8, 8), 2, "gather", False),
    ((30, 448, 48, 8, 8), 2, "pointwise", False),       # ... nor where the gather would share out its channels
    # pooled on the way: only with enough workgroups for the length of the sum
    ((16, 803, 73, 16, 16), 2, "gather", False),
    ((127, 803, 73, 16, 16), 2, "gather", False),
    ((128, 803, 73, 16, 16), 2, "pointwise", True),
    ((32, 201, 73, 16, 16), 2, "gather", False),
    ((64, 201, 73, 16, 16), 2, "pointwise", True),
    ((31, 201, 73, 12, 12), 2, "gather", False),
    ((32, 201, 73, 12, 12), 2, "pointwise", True),
    ((32, 190, 73, 16, 16), 2, "pointwise", True),
    # ... more of them where a second tile of output channels pools the same input once more
    ((63, 201, 64, 16, 16), 2, "gather", False),
    ((64, 201, 64, 16, 16), 2, "pointwise", True),
    ((31, 201, 64, 12, 12), 2, "pointwise", True),
    ((60, 201, 73, 16, 16), 2, "gather", False),
    ((60, 200, 73, 16, 16), 2, "pointwise", True),      # (rows of W that are whole items)
    ((64, 803, 64, 16, 16), 2, "pointwise", True),
    ((127, 1300, 64, 16, 16), 2, "gather", False),
    ((128, 1300, 64, 16, 16), 2, "pointwise", True),
    # ... and not by the few threads that have channels to move
    ((198, 10, 14, 68, 68), 2, "pointwise", False),
    ((20, 10, 14, 68, 68), 2, "pointwise", True),
    ((198, 33, 14, 68, 68), 2, "pointwise", True),
    # rows that the gather's LDS has no room for stay
    ((1, 16, 16, 2, 504), 2, "pointwise", False),
    ((1, 700, 16, 3, 1000), 1, "pointwise", False),
    ((2, 700, 16, 8, 104), 2, "gather", False),
    # planes of two or four pixels
    ((199, 864, 1295, 2, 2), 4, "gather", False),
    ((199, 864, 1295, 3, 2), 4, "pointwise", False),
    ((512, 2048, 1000, 1, 1), 1, "pointwise", False),
])
def test_pointwise_layers(shape, k, plan, pooled):
    d = B.make_desc(*shape, 1, 1, pool_kh=k, pool_kw=k)
    got = B.cac_describe_plan(d, B.OP_FWD_AND_COMPRESS)
    assert got.startswith(plan) and ("pooled on the way" in got) == pooled, got


@pytest.mark.parametrize("shape,kh,plan", [
    # N, C, K, H, W.  3 x 3 stride-2 weight gradient from tiles of one column: the split of the copy registers that gives long
    # rows two output rows per chunk does not fit the 64 x 64 tile there; the 32 x 32 one only where it has no more to copy
    ((20, 312, 899, 73, 73), 1, "variant=2 tile=64x64 chunk=1img x 1rows"),
    ((10, 1037, 168, 103, 103), 2, "variant=2 tile=64x64 chunk=1img x 1rows"),
    ((500, 145, 817, 2, 68), 1, "variant=2 tile=64x64 chunk=1img x 1rows"),
    ((185, 28, 19, 161, 76), 1, "variant=3 tile=32x32 chunk=1img x 2rows"),
    ((112, 11, 103, 73, 73), 1, "variant=3 tile=32x32 chunk=1img x 2rows"),
    ((25, 544, 637, 54, 54), 1, "variant=2 tile=64x64 chunk=1img x 2rows"),
    # ... and the first split, where a workgroup has eight to eleven chunks, only in the same tile and for fewer chunks
    ((421, 3, 536, 18, 18), 8, "variant=3 tile=32x32 chunk=3img x 9rows"),
    ((11, 400, 368, 40, 40), 8, "variant=3 tile=32x32 chunk=1img x 20rows"),
    ((112, 614, 3, 5, 198), 8, "passes dy=8"),
    ((27, 444, 398, 25, 3), 1, "passes dy=4"),
    ((3, 179, 1397, 6, 79), 1, "passes dy=4"),
])
def test_stride2_weight_gradient_from_tiles_of_one_column(shape, kh, plan):
    d = B.make_desc(*shape, 3, 3, 2, 2, 1, 1, kh, 1, dtype=B.BF16)
    got = B.cac_describe_plan(d, B.OP_BWD_WEIGHT_COMPRESSED)
    assert plan in got, got


@pytest.mark.parametrize("shape,k,waves", [
    # N, C, K, H, W.  1 x 1: the waves of their own give way where 385 to 512 workgroups of the other kernel hold little padding ...
    ((15, 816, 1824, 5, 43), 4, 0),
    ((5, 866, 1280, 29, 38), 1, 0),
    ((255, 128, 128, 13, 32), 4, 0),
    ((114, 35, 141, 39, 11), 1, 1),       # ... but not to a quarter of it,
    ((13, 816, 1824, 5, 43), 4, 4),       # to fewer workgroups,
    ((259, 128, 128, 13, 32), 4, 1),      # to more,
    ((45, 2048, 320, 22, 22), 1, 4),      # with four waves to a tile to few tiles of channels,
    ((30, 96, 256, 33, 41), 4, 1),        # nor with one on planes of an odd size
    ((64, 512, 2048, 7, 7), 2, 0),
    ((64, 2048, 512, 7, 7), 2, 4),
])
def test_pointwise_layers_by_waves(shape, k, waves):
    d = B.make_desc(*shape, 1, 1, pool_kh=k, pool_kw=k)
    got = B.cac_describe_plan(d, B.OP_FWD_AND_COMPRESS)
    assert got.startswith("pointwise") and (f"waves/tile={waves}" if waves else "img/tile") in got, got


@pytest.mark.parametrize("shape,pixels", [
    # N, C, K, H, W.  1 x 1, odd planes: tiles of whole images are for four waves to a tile
    ((124, 128, 1648, 7, 7), "56px ch/pass=64 waves/tile=1"),
    ((171, 32, 1104, 3, 15), "56px ch/pass=64 waves/tile=1"),
    ((420, 64, 912, 5, 7), "56px ch/pass=64 waves/tile=1"),
    ((32, 256, 1024, 7, 7), "49px ch/pass=64 waves/tile=4"),
    ((13, 264, 392, 5, 5), "50px ch/pass=64 waves/tile=4"),
])
def test_pointwise_wave_tiles_of_odd_planes(shape, pixels):
    d = B.make_desc(*shape, 1, 1, pool_kh=2, pool_kw=2)
    got = B.cac_describe_plan(d, B.OP_FWD_AND_COMPRESS)
    assert got.startswith("pointwise by waves tile=64ch x " + pixels), got


@pytest.mark.parametrize("shape,waves", [
    # N, C, K, H, W.  3 x 3 stride 2, few workgroups: the gather shares long sums out, six stages a wave and more
    ((2, 592, 27, 5, 48), False),
    ((2, 592, 27, 5, 47), True),       # ... not where its copy of the input moves single elements,
    ((2, 320, 27, 5, 48), True),       # nor up to five stages
    ((2, 321, 27, 5, 48), False),
    ((4, 592, 300, 5, 48), False),
    ((5, 592, 400, 5, 48), True),      # nor past 32 workgroups
    ((1, 704, 27, 5, 47), True),      # from twelve stages on wherever it can
    ((1, 705, 27, 5, 47), False),
])
def test_long_sums_of_stride_2_layers(shape, waves):
    got = B.cac_describe_plan(B.make_desc(*shape, 3, 3, 2, 2, 1, 1), B.OP_FWD_AND_COMPRESS)
    assert ("by waves" in got) == waves and got.startswith("gather") != waves, got


@pytest.mark.parametrize("shape,op,waves", [
    # N, C, K, H, W.  3 x 3 stride 1, rows that give a lane two items a stage: the line to the large tiles lies lower
    ((7, 67, 464, 51, 51), B.OP_BWD_DATA, False),
    ((30, 176, 118, 5, 47), B.OP_BWD_DATA, True),
    ((39, 725, 19, 23, 47), B.OP_FWD_AND_COMPRESS, False),
    ((9, 560, 148, 20, 55), B.OP_FWD_AND_COMPRESS, True),
    # ... and few workgroups with long sums leave them to the gather, as under stride 2
    ((2, 32, 1344, 16, 47), B.OP_BWD_DATA, False),
    ((2, 32, 1344, 15, 47), B.OP_BWD_DATA, True),
    ((2, 32, 1344, 16, 39), B.OP_BWD_DATA, True),
])
def test_two_items_to_a_lane(shape, op, waves):
    got = B.cac_describe_plan(B.make_desc(*shape, 3, 3, 1, 1, 1, 1), op)
    assert ("by waves" in got) == waves, got


@pytest.mark.parametrize("shape,stride,op,lds", [
    # N, C, K, H, W.  1 x 1 in float: the plain kernel keeps data gradients of few outputs ...
    ((1, 54, 20, 14, 32), 1, B.OP_BWD_DATA, False),
    ((1, 54, 20, 14, 32), 2, B.OP_BWD_DATA, False),
    ((2, 102, 48, 26, 26), 1, B.OP_BWD_DATA, True),
    ((12, 144, 30, 73, 73), 1, B.OP_BWD_DATA, False),   # (... further on with four pixels per thread)
    ((21, 107, 59, 53, 53), 1, B.OP_BWD_DATA, True),
    # ... and strides past 2 are none of its business
    ((4, 16, 19, 13, 17), 3, B.OP_FWD_AND_COMPRESS, True),
])
def test_pointwise_float_layers(shape, stride, op, lds):
    got = B.cac_describe_plan(B.make_desc(*shape, 1, 1, stride, stride, dtype=B.F32), op)
    assert got.startswith("conv_lds") == lds, got


@pytest.mark.parametrize("shape,stride,op,waves", [
    # N, C, K, H, W.  3 x 3 layers that only the waves take with matrix instructions: not where a launch without any is faster
    ((6, 3, 3, 1, 1), 1, B.OP_BWD_DATA, False),
    ((2, 52, 1, 1, 1), 1, B.OP_BWD_DATA, False),
    ((7, 5, 259, 1, 1), 1, B.OP_BWD_DATA, True),
    ((72, 21, 6, 2, 1), 1, B.OP_FWD_AND_COMPRESS, True),
    ((228, 2, 1, 42, 42), 2, B.OP_FWD_AND_COMPRESS, False),
    ((3, 2, 6, 5, 3), 2, B.OP_FWD_AND_COMPRESS, False),
    ((156, 178, 57, 4, 4), 2, B.OP_FWD_AND_COMPRESS, True),
    ((90, 29, 27, 3, 3), 2, B.OP_FWD_AND_COMPRESS, True),
])
def test_layers_of_few_terms_go_without_matrix_instructions(shape, stride, op, waves):
    got = B.cac_describe_plan(B.make_desc(*shape, 3, 3, stride, stride, 1, 1), op)
    assert ("by waves" in got) == waves and got.startswith(("conv_lds", "generic")) != waves, got
