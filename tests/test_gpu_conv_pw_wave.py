"""GPU parity of the 1 x 1 kernel whose waves stage for themselves: planes of odd size with tiles of whole images (49, 25 and 5
pixels) and with items that run from image to image (63 and 81), stores of 1 to 8 pixels, ragged channels on both sides,
sums whose stages do not divide among the four waves, a last tile with few images; one wave to a tile."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2409_11902_amd import binding as B
from paper_2409_11902_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    # N, C, K, H, W, waves to a tile (forward, data gradient; 0: another kernel)
    (5, 512, 328, 7, 7, 4, 4),       # whole images, 16-byte runs
    (5, 330, 300, 7, 7, 4, 4),       # K no multiple of 8 (forward), C neither (data gradient)
    (13, 264, 392, 5, 5, 4, 4),      # two images to a tile
    (37, 256, 264, 1, 5, 4, 4),      # eight images to a tile
    (3, 300, 520, 7, 9, 4, 4),       # more than a tile of odd pixels
    (3, 264, 256, 9, 9, 4, 4),
    (9, 650, 260, 4, 4, 4, 4),       # eight pixels per store
    (9, 260, 650, 6, 6, 4, 4),       # four
    (9, 260, 330, 5, 6, 4, 4),       # two, an item's last pixels in the next plane
    (1, 1500, 520, 2, 4, 4, 4),      # one item per image, fewer items than a tile has
    (1400, 72, 100, 7, 7, 1, 1),     # one wave to a tile, whole pieces of output channels or not
    (130, 40, 1104, 3, 15, 1, 4),
    (1500, 40, 136, 6, 6, 1, 0),
    (700, 260, 450, 9, 7, 1, 0),
]


@pytest.mark.parametrize("case", CASES, ids=[str(c[:5]) for c in CASES])
def test_step(case):
    from gpu_util import run_step
    N, C, K, H, W, fwd, dx = case
    spec = synth.LayerSpec(f"pw-wave-{N}-{C}-{K}-{H}-{W}", N, C, K, H, W, R=1, S=1, pad=0)
    t = synth.make_inputs(spec, "pw-wave")
    d = B.desc_from_spec(spec)
    for op, n in ((B.OP_FWD_AND_COMPRESS, fwd), (B.OP_BWD_DATA, dx)):
        plan = B.cac_describe_plan(d, op)
        assert ("by waves" in plan) == bool(n) and (not n or f"waves/tile={n}" in plan), plan
    got = run_step(spec, t)
    w = t["W"].astype(np.float64).reshape(K, C)
    x, dy = (t[n].astype(np.float64).reshape(N, -1, H * W) for n in ("X", "dY"))
    y = np.matmul(w, x) + t["b"].astype(np.float64).reshape(1, K, 1)
    # float sums of at most 1500 terms (2e-6 of the norm), then one rounding to bfloat16: 2^-9 of a value at most
    for name, want in (("Y", y), ("dX", np.matmul(w.T, dy))):
        a = got[name].reshape(want.shape)
        scale = np.sqrt(np.mean(want ** 2))
        assert np.all(np.abs(a - want) <= 2.0 ** -8 * np.abs(want) + 2e-5 * scale), name
    assert np.allclose(got["Z"], oracle.avgpool(t["X"].astype(np.float64), spec.k, spec.k), rtol=2.0 ** -7, atol=1e-6)
