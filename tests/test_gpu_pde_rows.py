"""Laplacian rows at the edges of the assembly's ways, against the oracle.

A vertex holds eight triangles in place (more are chained: up to 32 a wave's
lanes work the row out, beyond that one lane), rows are worked out 64 at a
time in LDS room for 512 entries, and laid out in slices of 16.  Every sum has
one stated order on both sides, so the operator, K u and the heat steps are
identical bit for bit.
"""
from __future__ import annotations

import math

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _fans(degrees, rs):
    """Closed fans of the given numbers of triangles, their triangles shuffled."""
    v, t = [], []
    for n, d in enumerate(degrees):
        c = len(v)
        v.append((4.0 * n, 0.0))
        v += [(4.0 * n + math.cos(2 * math.pi * k / d), math.sin(2 * math.pi * k / d)) for k in range(d)]
        t += [(c, c + 1 + k, c + 1 + (k + 1) % d) for k in range(d)]
    return np.array(v), np.array(t, np.int32)[rs.permutation(len(t))]


def _random(nv, nt, rs):
    """Triangles of random vertices (non-manifold, of any degree), positively oriented."""
    p = rs.uniform(0, 10, (nv, 2))
    t = rs.integers(0, nv, (nt, 3)).astype(np.int32)
    a, b, c = p[t[:, 0]], p[t[:, 1]], p[t[:, 2]]
    area = (b[:, 0] - a[:, 0]) * (c[:, 1] - a[:, 1]) - (b[:, 1] - a[:, 1]) * (c[:, 0] - a[:, 0])
    t[area < 0] = t[area < 0][:, [0, 2, 1]]
    return p, t[area != 0]


CASES = {
    "fans around the slots": lambda rs: _fans([3, 6, 7, 8, 9, 10, 8, 9], rs),
    "fans around a wave": lambda rs: _fans([31, 32, 33, 40, 6, 64, 65], rs),
    "one row more than a wave, full rows": lambda rs: _random(65, 170, rs),
    "more than the staged entries": lambda rs: _random(250, 640, rs),
    "one block less one": lambda rs: _random(255, 500, rs),
    "one block and one": lambda rs: _random(257, 1100, rs),
    "nearly all chained": lambda rs: _random(300, 4000, rs),
    "far apart ids": lambda rs: _random(40000, 30000, rs),
}


@pytest.mark.parametrize("name", list(CASES))
def test_rows_match_oracle(name):
    import torch

    from paper_2602_19474_amd.pde import Laplacian
    rs = np.random.default_rng(sorted(CASES).index(name))
    v, t = CASES[name](rs)
    print(f"[gpu-pde-rows] {name}: {len(v)} vertices, {len(t)} triangles", flush=True)
    lap = Laplacian(torch.from_numpy(v).cuda(), torch.from_numpy(t).cuda())
    ref = oracle.laplacian(v, t)
    c = lap.csr()
    for key in ("row_off", "col", "val", "mass"):
        assert np.array_equal(c[key].cpu().numpy(), ref[key]), key
    assert np.array_equal(c["boundary"].cpu().numpy().astype(bool), ref["boundary"])
    for key in ("nnz", "n_boundary", "n_invalid", "min_mass", "lambda_bound"):
        assert lap.info[key] == ref[key], key
    u = rs.standard_normal(len(v))
    assert np.array_equal(lap.apply(torch.from_numpy(u).cuda()).cpu().numpy(), oracle.laplacian_apply(v, t, u))
    dt = 1.9 / (500.0 * ref["lambda_bound"])
    ug = torch.from_numpy(u).cuda()
    lap.heat_steps(ug, 500.0, dt, 3)
    # a vertex in no triangle has no mass: its steps are NaN (0 / 0) on both sides
    assert np.array_equal(ug.cpu().numpy(), oracle.heat_steps(v, t, u, 500.0, dt, 3), equal_nan=True)
