"""The mesh of Alg. 3 where the ways of the probe and of the cut triangles meet.

Cut grid triangles have room for one in sixteen owners (at least 65536): on
bitmaps of fine noise most have none and take the general subdivision, beside
neighbours that were kept, and both write the crossings of their common edges.
Small and thin images hold owners at the grid's border and with split sides,
which the probe takes one by one beside the plain ones.
"""
from __future__ import annotations

import pytest

from paper_2602_19474_amd import workloads as wl
from test_gpu_preprocess_mesh import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size,sigma,h", [(900, 2.0, 1), (1000, 3.0, 2)])
def test_more_cut_triangles_than_room(size, sigma, h):
    bm = wl.smoothed_noise(size, size, sigma, 0.0, False, wl.rng(9, 1))
    m = _compare(f"noise{size} sigma {sigma}", bm, h)
    assert m.n_cut > 65536


@pytest.mark.parametrize("w,h", [(3, 40), (40, 3), (17, 65), (65, 17), (64, 64)])
def test_border_owners(w, h):
    _compare(f"noise {w}x{h}", wl.smoothed_noise(w, h, 1.5, 0.0, False, wl.rng(9, w)), 1)
