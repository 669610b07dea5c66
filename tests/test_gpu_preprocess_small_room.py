"""The mesh of Alg. 3 on small images, where cut triangles have two slots for each
owner: boards of single samples, which cut more triangles than any other picture."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_preprocess_mesh import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,grid_h,s", [(2, 2, 1, 2), (16, 16, 1, 2), (64, 64, 1, 2), (65, 33, 2, 3), (40, 40, 0.5, 1)])
def test_boards(w, h, grid_h, s):
    y, x = np.mgrid[0:h, 0:w]
    _compare(f"board {w}x{h}", ((x // s + y // s) % 2).astype(np.uint8), grid_h)
