"""Alg. 3 where the row segments of its passes end: grids of a few owners more and
fewer than a wave's 64 and a segment's 256, narrow ones whose rows share a word of
the vertex compaction, and fine noise, where most owners have a moved corner or a
split side.  The grid and its mesh against the oracle.
"""
from __future__ import annotations

import pytest

from paper_2602_19474_amd import workloads as wl
from test_gpu_preprocess import _compare as compare_grid
from test_gpu_preprocess_mesh import _compare as compare_mesh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w", [1, 2, 7, 29, 59, 61, 62, 125, 252, 253, 255, 509])
@pytest.mark.parametrize("sigma", [1.0, 6.0])
def test_row_ends(w, sigma):
    bm = wl.smoothed_noise(w, 37, sigma, 0.0, False, wl.rng(11, w))
    compare_grid(f"{w} columns", bm, 1)
    compare_mesh(f"{w} columns", bm, 1)
