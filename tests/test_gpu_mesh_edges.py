"""Meshing where its kernels and launches change: calls of as many owner rows as
a dispatch rule's line lies at and of one more, coarsening from rows of every
alignment, and batches around the 64 images that one look at a block table
compares.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_2602_19474_amd as sbmt
from paper_2602_19474_amd import workloads as wl
from paper_2602_19474_amd.batch import mesh_batch
from test_gpu_parity import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [2048, 4096, 8192, 32768])
@pytest.mark.parametrize("more", [False, True])
def test_rows_at_a_rules_line(rows, more):
    hi = rows
    while sbmt.query(12, hi, 1).grid_rows <= rows:
        hi += 1
    while sbmt.query(12, hi - 1, 1).grid_rows > rows:
        hi -= 1
    h = hi if more else hi - 1  # the least height of more rows, the largest of at most so many
    bm = (wl.rng(5, rows).random((h, 12)) < 0.5).astype(np.uint8)
    _compare(f"{rows} rows, more={more}", bm, 1, check_invariants=False)


@pytest.mark.parametrize("h", [0.5, 1, 2, 2.5, 3, 4, 4.5, 5, 6])
@pytest.mark.parametrize("x0,y0,w", [(0, 0, 1040), (5, 3, 777), (16, 1, 1), (15, 0, 18)])
def test_coarsening_of_views(h, x0, y0, w):
    import torch
    full = (wl.rng(6, int(2 * h)).random((70, 1061)) < 0.5).astype(np.uint8) * 255
    view = torch.from_numpy(full).cuda()[y0:, x0:x0 + w]
    v, t, c = sbmt.mesh_from_bitmap(view, h)
    ref = oracle.mesh_from_bitmap(np.ascontiguousarray(full[y0:, x0:x0 + w]), h)
    assert np.array_equal(t.cpu().numpy(), ref.tris) and np.array_equal(c.cpu().numpy(), ref.codes)
    assert float(np.abs(v.cpu().numpy() - ref.verts).max(initial=0.0)) <= 1e-12 * h


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 128, 4097])
def test_batches_around_one_look_at_the_table(n):
    import torch
    g = wl.rng(7, n)
    shapes = [(9, 7), (1, 30), (0, 0), (25, 18), (40, 3)]
    bms = [(g.random(s) < 0.6).astype(np.uint8) for s in shapes]
    refs = [oracle.mesh_from_bitmap(b, 1) for b in bms]
    dev = [torch.from_numpy(b).cuda() for b in bms]
    outs = mesh_batch([(dev[i % 5], 1) for i in range(n)])
    assert len(outs) == n
    for i, (v, t, c) in enumerate(outs):
        ref = refs[i % 5]
        assert tuple(t.shape) == ref.tris.shape, (n, i)
        if i % 97 < 5 or i >= n - 5:
            assert np.array_equal(t.cpu().numpy(), ref.tris) and np.array_equal(c.cpu().numpy(), ref.codes), (n, i)
            assert float(np.abs(v.cpu().numpy() - ref.verts).max(initial=0.0)) <= 1e-12, (n, i)


@pytest.mark.parametrize("sides", [(0, 1), (1, 0, 0, 0), (0, 0, 0), (1, 1, 1)])
@pytest.mark.parametrize("tile_rows", [4, 8, 16])
def test_batches_of_one_side_and_of_both(sides, tile_rows, monkeypatch):
    import torch
    from paper_2602_19474_amd.batch import Tuning
    bms = [wl.smoothed_noise(90 + 130 * i, 75, 5.0, 0.0, False, wl.rng(8, i)) for i in range(len(sides))]
    make, left = sbmt._image, list(sides)
    monkeypatch.setattr(sbmt, "_image", lambda t, h, flags: make(t, h, left.pop(0)))
    outs = mesh_batch([(torch.from_numpy(b).cuda(), 1) for b in bms], tuning=Tuning(strategy=0, tile_rows=tile_rows))
    for i, (v, t, c) in enumerate(outs):
        ref = oracle.mesh_from_bitmap(bms[i], 1, oracle.BOTH_SIDES if sides[i] else 0)
        assert np.array_equal(t.cpu().numpy(), ref.tris) and np.array_equal(c.cpu().numpy(), ref.codes), (sides, i)
        assert float(np.abs(v.cpu().numpy() - ref.verts).max(initial=0.0)) <= 1e-12, (sides, i)


@pytest.mark.parametrize("h", [0.5, 1, 1.5, 2.5, 3, 5, 6])
def test_coarsening_of_many_blocks(h):
    import torch
    g = wl.rng(9, int(2 * h))
    bms = [(g.random(s) < 0.5).astype(np.uint8) for s in [(37, 700), (5, 1), (71, 90)]]
    dev = [torch.from_numpy(b).cuda() for b in bms]
    outs = mesh_batch([(dev[i % 3], h) for i in range(2600)])
    refs = [oracle.mesh_from_bitmap(b, h) for b in bms]
    for i in [*range(7), *range(1000, 1012), *range(2590, 2600)]:
        v, t, c = outs[i]
        assert np.array_equal(t.cpu().numpy(), refs[i % 3].tris) and np.array_equal(c.cpu().numpy(), refs[i % 3].codes)
        assert float(np.abs(v.cpu().numpy() - refs[i % 3].verts).max(initial=0.0)) <= 1e-12 * h
