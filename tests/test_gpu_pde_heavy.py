"""Laplacian rows of many triangles against the oracle, identical bit for bit.

A vertex of more than eight triangles is worked out by a wave, 64 candidate
neighbours (of 32 triangles) at a time, its list sorted in place up to 64
triangles and through scratch memory beyond: closed fans at and around those
numbers, and triangles of random vertices, whose rows hold every neighbour
several times, in other chunks of candidates too.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from test_gpu_pde_rows import _fans, _random

pytestmark = pytest.mark.gpu

CASES = {
    "fans around the chunks": lambda rs: _fans([31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 500], rs),
    "repeated neighbours, 40 a vertex": lambda rs: _random(30, 400, rs),
    "repeated neighbours, 200 a vertex": lambda rs: _random(60, 4000, rs),
    "of every size": lambda rs: _random(900, 30000, rs),
}


@pytest.mark.parametrize("name", list(CASES))
def test_rows_of_many_triangles(name):
    import torch

    from paper_2602_19474_amd.pde import Laplacian
    rs = np.random.default_rng(11 + sorted(CASES).index(name))
    v, t = CASES[name](rs)
    print(f"[gpu-pde-heavy] {name}: {len(v)} vertices, {len(t)} triangles", flush=True)
    ref = oracle.laplacian(v, t)
    lap = Laplacian(torch.from_numpy(v).cuda(), torch.from_numpy(t).cuda())
    c = lap.csr()
    for key in ("row_off", "col", "val", "mass"):
        assert np.array_equal(c[key].cpu().numpy(), ref[key]), key
    assert np.array_equal(c["boundary"].cpu().numpy().astype(bool), ref["boundary"])
    for key in ("nnz", "n_boundary", "n_invalid", "min_mass", "lambda_bound"):
        assert lap.info[key] == ref[key], key
