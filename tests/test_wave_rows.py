"""Host-only: the rows that a tile of csrc/conv_wave.hip stages are those that the taps of its pixels meet, over random layers
(tests/host/wave_rows_walk.cpp, compiled with the header that the kernels use)."""
from __future__ import annotations

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("wave_rows") / "walk")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_2409_11902_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "wave_rows_walk.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("taps,stride,pad", [
    (3, 1, 3), (3, 2, 3), (9, 1, 9), (9, 2, 9), (1, 1, 1),
    # padding above the filter's height: a tile may start below its image's last row
    (3, 1, 14), (3, 2, 14), (9, 1, 14), (9, 2, 14), (1, 1, 14),
    # a filter flatter than the stride
    (1, 2, 1), (1, 2, 14),
])
def test_a_tile_stages_the_rows_that_its_taps_meet(walk, taps, stride, pad):
    r = subprocess.run([walk, str(taps), str(stride), str(pad), "2000"], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
