"""The CSR arrays that a Laplacian hands out are the ones it applies."""
from __future__ import annotations

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def test_apply_reads_the_arrays_csr_hands_out():
    """A weight changed through the view is the one that the next apply uses: K u
    of the changed rows, each summed in row order."""
    import torch

    from paper_2602_19474_amd import workloads as wl
    from paper_2602_19474_amd.pde import Laplacian
    print("[gpu-pde-views] apply after a change through csr()", flush=True)
    m = oracle.mesh_from_bitmap(wl.ellipses(120, 90, g=wl.rng(3, 1)), 1)
    lap = Laplacian(torch.from_numpy(m.verts).cuda(), torch.from_numpy(m.tris).cuda())
    c = lap.csr()
    u = np.random.default_rng(5).standard_normal(len(m.verts))
    c["val"].mul_(-2.0)  # exact, so that the sums are exactly doubled and turned
    y = lap.apply(torch.from_numpy(u).cuda()).cpu().numpy()
    assert np.array_equal(y, -2.0 * oracle.laplacian_apply(m.verts, m.tris, u))
    c["val"].mul_(-0.5)
    c["val"][0] = 7.0  # one entry of row 0
    off, col, val = (c[k].cpu().numpy() for k in ("row_off", "col", "val"))
    row0 = 0.0
    for e in range(off[0], off[1]):
        row0 = row0 + val[e] * (u[0] - u[col[e]])
    y = lap.apply(torch.from_numpy(u).cuda()).cpu().numpy()
    assert y[0] == row0 and np.array_equal(y[1:], oracle.laplacian_apply(m.verts, m.tris, u)[1:])
