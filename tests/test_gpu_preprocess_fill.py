"""sbmt_preprocess_mesh_fill through the C ABI: what it writes of a counted mesh,
and the workspaces and arguments it refuses without touching an output."""
from __future__ import annotations

import ctypes

import pytest

from paper_2602_19474_amd import workloads as wl

pytestmark = pytest.mark.gpu


class _Call:
    """An image with a workspace, and outputs of one spare row past `nv`, `nt` that hold sentinels."""

    def __init__(self, bitmap, grid_h):
        import torch

        from paper_2602_19474_amd import _image, _lib, context
        from paper_2602_19474_amd.preprocess import paper_thresholds, preprocess_mesh
        self.L, self.h = _lib.lib(), context(0).handle
        self.bm = torch.from_numpy(bitmap).to("cuda")
        self.img = _image(self.bm, grid_h, 0)
        self.th = paper_thresholds(grid_h)
        self.ref = preprocess_mesh(self.bm, grid_h)
        self.nv, self.nt = self.ref.verts.shape[0], self.ref.tris.shape[0]
        b, g = ctypes.c_size_t(), ctypes.c_int64()
        assert self.L.sbmt_pre_mesh_query(ctypes.byref(self.img), ctypes.byref(b), ctypes.byref(g)) == 0
        self.bytes = int(b.value)
        self.counts = (ctypes.c_int64 * 8)()
        self.verts = torch.empty((self.nv + 1, 2), dtype=torch.float64, device="cuda")
        self.tris = torch.empty((self.nt + 1, 3), dtype=torch.int32, device="cuda")
        self.codes = torch.empty((self.nt + 1,), dtype=torch.uint8, device="cuda")

    def clear(self):
        self.verts.fill_(-7.0)
        self.tris.fill_(-7)
        self.codes.fill_(7)

    def untouched(self, nv=0, nt=0):
        return (bool((self.verts[nv:] == -7.0).all()) and bool((self.tris[nt:] == -7).all())
                and bool((self.codes[nt:] == 7).all()))

    def call(self, fn, ws, vcap, tcap, th=None, nbytes=None):
        from paper_2602_19474_amd import _stream_ptr
        return getattr(self.L, fn)(self.h, ctypes.byref(self.img), *(th or self.th), ws.data_ptr(),
                                   self.bytes if nbytes is None else nbytes, self.verts.data_ptr(), vcap,
                                   self.tris.data_ptr(), self.codes.data_ptr(), tcap, self.counts, _stream_ptr(None))

    def size(self, ws):
        from paper_2602_19474_amd import _stream_ptr
        return self.L.sbmt_preprocess_mesh(self.h, ctypes.byref(self.img), *self.th, ws.data_ptr(), self.bytes, None, 0,
                                           None, None, 0, self.counts, _stream_ptr(None))

    def fill(self, ws, vcap=None, tcap=None, **kw):
        return self.call("sbmt_preprocess_mesh_fill", ws, self.nv if vcap is None else vcap,
                         self.nt if tcap is None else tcap, **kw)

    def filled(self):
        import torch
        return (torch.equal(self.verts[:self.nv], self.ref.verts) and torch.equal(self.tris[:self.nt], self.ref.tris)
                and torch.equal(self.codes[:self.nt], self.ref.codes) and self.untouched(self.nv, self.nt)
                and tuple(self.counts) == (self.nv, self.nt, self.ref.n_snapped, self.ref.n_repelled,
                                           self.ref.n_inserted, 0, self.ref.n_grid_vertices, self.ref.n_cut))


# ordinary shapes; noise with cut triangles beyond their slots (the general
# subdivision writes those)
@pytest.mark.parametrize("name", ["ellipses", "noise"])
def test_fill_writes_the_counted_mesh(name):
    import torch
    print(f"[gpu-pre-fill] {name}", flush=True)
    noise = name == "noise"
    c = _Call(wl.smoothed_noise(900, 900, 2.0, 0.0, False, wl.rng(9, 1)) if noise else
              wl.ellipses(150, 130, g=wl.rng(91, 4)), 1)
    assert not noise or c.ref.n_cut > 65536
    ws = torch.empty(c.bytes, dtype=torch.uint8, device="cuda")
    assert c.size(ws) == -7
    for _ in range(2):  # the counted mesh, as often as asked for
        c.clear()
        assert c.fill(ws) == 0 and c.filled()
    for vcap, tcap in ((0, 0), (c.nv - 1, c.nt), (c.nv, c.nt - 1), (c.nv // 2, c.nt // 3)):
        c.clear()
        assert c.fill(ws, vcap, tcap) == -7, (vcap, tcap)
        assert (c.counts[0], c.counts[1], c.counts[5]) == (c.nv, c.nt, -7)
        assert c.untouched(vcap, tcap)
    c.clear()
    assert c.fill(ws) == 0 and c.filled()
    # after a call that wrote less than it counted, and after one that wrote all
    for vcap, tcap, st in ((c.nv // 2, c.nt // 3, -7), (c.nv, c.nt, 0)):
        assert c.call("sbmt_preprocess_mesh", ws, vcap, tcap) == st
        c.clear()
        assert c.fill(ws) == 0 and c.filled()
    # refused before any launch
    c.clear()
    for th in ((0.4, 0.2, 0.1), (0.4, 0.1, 0.29), (0.5, 0.1, 0.1), (-0.1, 0.0, 0.0)):
        assert c.fill(ws, th=th) == -1, th
    assert c.fill(ws, nbytes=c.bytes - 1) == -4
    assert c.fill(ws, vcap=-1) == -1 and c.untouched()


def test_fill_refuses_a_workspace_without_its_plan():
    """The passes that write follow indices from the workspace, so none may run
    over memory that does not hold this image's plan."""
    import torch

    import paper_2602_19474_amd as sbmt
    from paper_2602_19474_amd.preprocess import Preprocessor
    print("[gpu-pre-fill] workspaces without the plan", flush=True)
    c = _Call(wl.ellipses(150, 130, g=wl.rng(91, 4)), 1)
    other = _Call(wl.ellipses(131, 150, g=wl.rng(91, 5)), 1)
    ws = torch.empty(max(c.bytes, other.bytes), dtype=torch.uint8, device="cuda")

    def refused(**kw):
        c.clear()
        return c.fill(ws, **kw) == -1 and c.untouched() and list(c.counts) == [0, 0, 0, 0, 0, -1, 0, 0]

    for byte in (0, 0xff, 0x5a):  # never planned
        ws.fill_(byte)
        assert refused(), byte
    assert other.size(ws) == -7  # another image's plan
    assert refused()
    assert c.size(ws) == -7  # this image's, other thresholds
    assert refused(th=tuple(0.5 * t for t in c.th))
    assert c.fill(ws) == 0 and c.filled()
    sbmt.plan(c.bm, 1, ws)  # other calls on the workspace since
    assert refused()
    assert c.size(ws) == -7
    p = Preprocessor(c.bm, 1)
    p.ws = ws
    p.run()
    assert refused()
    assert c.size(ws) == -7
    assert c.fill(ws) == 0 and c.filled()


@pytest.mark.parametrize("grid_h,size,seed", [(2.5, 150, 50), (2.5, 150, 51), (1.25, 75, 52)])
def test_a_plan_that_failed_is_not_written(grid_h, size, seed):
    """At these edges a polyline vertex can lie within b of two sides, which the
    oracle refuses, too.  The counts and numbers of such a plan do not fit
    together: no pass may write by them, in the call itself or in a fill."""
    import ctypes

    import torch

    import oracle
    from paper_2602_19474_amd import _image, _lib, _stream_ptr, context
    from paper_2602_19474_amd.preprocess import paper_thresholds
    print(f"[gpu-pre-fill] failed plan {size} h={grid_h} seed {seed}", flush=True)
    bm = wl.smoothed_noise(size, size, 6.0, 0.0, False, wl.rng(seed, int(grid_h * 64)))
    with pytest.raises(oracle.OracleError):
        oracle.mesh_preprocessed(bm, grid_h)
    t = torch.from_numpy(bm).to("cuda")
    L, h, img, th = _lib.lib(), context(0).handle, _image(t, grid_h, 0), paper_thresholds(grid_h)
    b, g = ctypes.c_size_t(), ctypes.c_int64()
    assert L.sbmt_pre_mesh_query(ctypes.byref(img), ctypes.byref(b), ctypes.byref(g)) == 0
    ws = torch.empty(int(b.value), dtype=torch.uint8, device="cuda")
    cap = 50000
    counts = (ctypes.c_int64 * 8)()
    verts = torch.full((cap, 2), -7.0, dtype=torch.float64, device="cuda")
    tris = torch.full((cap, 3), -7, dtype=torch.int32, device="cuda")
    codes = torch.full((cap,), 7, dtype=torch.uint8, device="cuda")
    for byte in (0, 0xff):  # whatever the workspace held
        ws.fill_(byte)
        for fn, st in (("sbmt_preprocess_mesh", -6), ("sbmt_preprocess_mesh_fill", -1)):
            assert getattr(L, fn)(h, ctypes.byref(img), *th, ws.data_ptr(), ws.numel(), verts.data_ptr(), cap,
                                  tris.data_ptr(), codes.data_ptr(), cap, counts, _stream_ptr(None)) == st
            assert counts[5] == st
    assert bool((verts == -7.0).all()) and bool((tris == -7).all()) and bool((codes == 7).all())
