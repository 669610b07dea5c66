"""Mesh quality at triangle counts where its passes' blocks and rounds end: one
workgroup's keys of a select pass, the first and second round of the quality
pass's and of a select pass's grid.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from test_gpu_post import _check_quality

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4096, 8191, 8192, 8193, 524288, 524289, 4_194_305])
def test_quality_counts(n):
    import torch

    from paper_2602_19474_amd.post import mesh_quality
    rs = np.random.default_rng(n)
    verts = rs.uniform(-20, 20, (max(3, n // 3), 2))
    tris = rs.integers(0, verts.shape[0], (n, 3)).astype(np.int32)
    tris[:: max(1, n // 50)] = tris[0]  # equal keys
    tris[rs.integers(1, n, 5), 1] = -1
    got = mesh_quality(torch.from_numpy(verts).cuda(), torch.from_numpy(tris).cuda(), allow_invalid=True)
    _check_quality(got, oracle.mesh_quality(verts, tris), verts, tris, f"{n} triangles")
