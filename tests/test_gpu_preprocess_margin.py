"""Steps 2 and 3 at thresholds next to a distance that occurs, against the oracle.

The distance that decides is a root of squares of whole coordinates, so it carries
their rounding (1e-12 px here), and a vertex is closer than a threshold by that
distance, not by a more exact one.  The image is 20040 px wide with shapes at its
far end; row 181 has vertices 0.00042290994695161983 px from 45 degree segments,
and row 104 sides that pass polyline vertices at 0.00017265226275606186 px.  Both
are nearer than the exact distance by more than a billionth of it.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2602_19474_amd import workloads as wl
from test_gpu_preprocess import _compare

pytestmark = pytest.mark.gpu


def _image():
    bm = np.zeros((172, 20040), np.uint8)
    bm[:, 19700:20000] = wl.smoothed_noise(300, 172, 2.0, 0.0, False, wl.rng(7, 3))
    return bm


@pytest.mark.parametrize("step,d,what", [("c", 0.00042290994695161983, "n_repelled"),
                                         ("b", 0.00017265226275606186, "n_inserted")])
def test_thresholds_next_to_a_distance(step, d, what):
    bm = _image()
    found = []
    for t in (d, float(np.nextafter(d, 1.0))):  # not closer than t, closer than t
        th = (2.2 * t, 0.0, t) if step == "c" else (2.2 * t, t, 0.0)
        _compare(f"threshold {step}", bm, 1, th)
        found.append(getattr(oracle.preprocessed_grid(bm, 1, *th), what))
    assert found[1] > found[0]
