"""Performance cases of the framework: what a program has it do, over the sizes it is used at.

``listed()`` names the cases, ``draw(rng)`` gives further ones of the same
ranges, ``prepare`` makes what a program holds before the call, ``run`` is one
pass through the public entry points, ``work`` the bytes and operations the
pass cannot do without and ``exact`` the computed outputs in plain 64-bit
torch.  Bitmaps follow the recipes of ``workloads.py`` (disks, ellipses,
smoothed noise), drawn on the GPU.

Kinds of case
  mesh    one bitmap to a mesh: ``call`` is ``from_bitmap`` (plan, allocate,
          run), ``plan_run`` (workspace and outputs kept by the program) or
          ``async`` (no host round trip)
  batch   many uneven bitmaps in one captured graph, replayed
  serve   a batch of requests: plan, allocate, emit
  grid    the preprocessed grid of Alg. 3, workspace and outputs kept
  alg3    the mesh of Alg. 3: ``call`` is ``once`` or ``kept``
  measure field sampling and quality statistics of a mesh
  laplace assembly of a mesh's cotangent Laplacian
  heat    a Gaussian pulse and explicit heat steps on an assembled mesh
"""
from __future__ import annotations

import math
import random

import torch

import paper_2602_19474_amd as sbmt
from paper_2602_19474_amd.batch import Batch, mesh_batch
from paper_2602_19474_amd.pde import Laplacian
from paper_2602_19474_amd.post import mesh_quality, sample_field
from paper_2602_19474_amd.preprocess import MeshPreprocessor, Preprocessor, preprocess_mesh

HALF_SQRT3 = 0.86602540378443864676
GRID_EDGES = (0.5, 0.75, 1.0, 1.5, 2.0, 3.0, 4.0)
LARGEST = 8192 * 8192  # lattice cells (pixels / h^2) of the largest listed case


def listed():
    return [
        # the smallest call: one disk, where launches and latency count
        {"name": "disk64", "kind": "mesh", "call": "from_bitmap", "w": 64, "h": 64, "edge": 1.0, "content": "disk",
         "both": False},
        # an ordinary picture of smooth shapes at a coarser grid
        {"name": "ellipses1024", "kind": "mesh", "call": "from_bitmap", "w": 1024, "h": 1024, "edge": 2.0,
         "content": "ellipses", "both": False},
        # a ragged image (unaligned rows, fractional edge, both sides) meshed without a host round trip
        {"name": "ragged_both", "kind": "mesh", "call": "async", "w": 2203, "h": 1531, "edge": 1.5,
         "content": "noise8", "both": True},
        # the largest single image, workspace and outputs kept by the program
        {"name": "noise8192", "kind": "mesh", "call": "plan_run", "w": 8192, "h": 8192, "edge": 1.0,
         "content": "noise16", "both": False},
        # many uneven images of a data set, one graph replay
        {"name": "batch64", "kind": "batch", "n": 64, "lo": 128, "hi": 2048},
        # one batch of a server's requests, log-uniform sides
        {"name": "serve12", "kind": "serve", "n": 12, "lo": 256, "hi": 4096},
        # the grid of Alg. 3 alone (a mesher that cuts it itself)
        {"name": "grid4000", "kind": "grid", "w": 4000, "h": 3000, "edge": 1.0, "content": "noise16"},
        # the mesh of Alg. 3: one call on an ordinary picture, and the largest one with everything kept
        {"name": "alg3_ellipses1024", "kind": "alg3", "call": "once", "w": 1024, "h": 1024, "edge": 2.0,
         "content": "ellipses"},
        {"name": "alg3_noise8192", "kind": "alg3", "call": "kept", "w": 8192, "h": 8192, "edge": 1.0,
         "content": "noise16"},
        # a mesh measured: a field brought onto it, its quality reported
        {"name": "measure4096", "kind": "measure", "w": 4096, "h": 4096, "edge": 1.0, "content": "noise16"},
        # a mesh made ready for a solver
        {"name": "laplace4096", "kind": "laplace", "w": 4096, "h": 4096, "edge": 1.0, "content": "noise16"},
        # a diffusion run on a mesh of bounded angles
        {"name": "heat2048", "kind": "heat", "w": 2048, "h": 2048, "edge": 1.0, "content": "noise8", "steps": 50},
    ]


def _log_int(rng: random.Random, lo: int, hi: int) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(("mesh", "mesh", "mesh", "batch", "serve", "grid", "alg3", "alg3", "measure", "laplace", "heat"))
    if kind == "batch":
        lo = _log_int(rng, 64, 512)
        return {"kind": kind, "n": rng.randint(4, 96), "lo": lo, "hi": rng.randint(2 * lo, 2048)}
    if kind == "serve":
        lo = _log_int(rng, 128, 512)
        return {"kind": kind, "n": rng.randint(1, 16), "lo": lo, "hi": rng.randint(2 * lo, 4096)}
    top = {"laplace": 4096, "heat": 3072}.get(kind, 8192)
    edge = rng.choice(GRID_EDGES)
    while True:
        w = _log_int(rng, 64 if edge <= 1.5 else 256, top)
        h = min(max(int(w * math.exp(rng.uniform(-1.0, 1.0))), 64), top)
        if w * h / (edge * edge) <= min(top * top, LARGEST):
            break
    case = {"kind": kind, "w": w, "h": h, "edge": edge, "content": rng.choice(("disk", "ellipses", "noise8", "noise16"))}
    if kind == "mesh":
        case["call"] = rng.choice(("from_bitmap", "plan_run", "async"))
        case["both"] = rng.random() < 0.2 and w * h / (edge * edge) <= LARGEST / 4
    elif kind == "alg3":
        case["call"] = "once" if w * h / (edge * edge) <= LARGEST / 4 and rng.random() < 0.5 else "kept"
    elif kind == "heat":
        case["steps"] = _log_int(rng, 1, 100)
    return case


# -- inputs -----------------------------------------------------------------------

def _device():
    return torch.device("cuda:0" if torch.cuda.is_available() else "cpu")


def _blur(x, sigma: float, dim: int):
    """Gaussian along one axis, truncated at 4 sigma, reflected at the ends."""
    n = x.shape[dim]
    r = min(int(4 * sigma), n - 1)
    wt = [math.exp(-0.5 * (j / sigma) ** 2) for j in range(-r, r + 1)]
    pad = torch.cat((x.narrow(dim, 0, r).flip(dim), x, x.narrow(dim, n - r, r).flip(dim)), dim)
    out = torch.zeros_like(x)
    for j, a in enumerate(wt):
        out.add_(pad.narrow(dim, j, n), alpha=a / sum(wt))
    return out


def _picture(w: int, h: int, content: str, gen: torch.Generator):
    dev = _device()
    if content.startswith("noise"):
        sigma = float(content[5:])
        x = torch.randn((h, w), generator=gen, device=dev)
        x = _blur(_blur(x, sigma, 1), sigma, 0)
        # 16: the large workload's threshold after z-normalisation; 8: half the area
        cut = (x.double().mean() + 0.3 * x.double().std()).float() if sigma == 16.0 else 0.0
        return (x > cut).to(torch.uint8)
    p = torch.rand((48, 5), generator=gen, device=dev, dtype=torch.float64).cpu().tolist()
    xx = torch.arange(w, device=dev, dtype=torch.float32)[None, :]
    yy = torch.arange(h, device=dev, dtype=torch.float32)[:, None]
    if content == "disk":
        cx, cy = (w - 1) / 2 + 4 * p[0][0] - 2, (h - 1) / 2 + 4 * p[0][1] - 2
        return ((xx - cx) ** 2 + (yy - cy) ** 2 <= (20.0 / 64.0 * min(w, h)) ** 2).to(torch.uint8)
    out = torch.zeros((h, w), dtype=torch.bool, device=dev)
    for u in p[:32]:
        a, b, th = 20 + 130 * u[2], 20 + 130 * u[3], math.pi * u[4]
        c, s = math.cos(th), math.sin(th)
        dx, dy = xx - u[0] * w, yy - u[1] * h
        out |= ((dx * c + dy * s) / a) ** 2 + ((dy * c - dx * s) / b) ** 2 <= 1.0
    for u in p[32:]:
        out ^= (xx - u[0] * w) ** 2 + (yy - u[1] * h) ** 2 <= (5 + 25 * u[2]) ** 2
    return out.to(torch.uint8)


def _stride(edge: float) -> int:
    """Coarse stride of a grid edge: the smallest s with s^2 > 2 edge^2."""
    s = 1
    while s * s <= 2 * edge * edge:
        s += 1
    return s


def _bitmap(w: int, h: int, edge: float, content: str, key: str, seed: int):
    """The bitmap of (key, seed).  The size of a mesh follows from its picture,
    and a case has one size: the picture is drawn from the key, and the seed
    arranges it anew (other vertices, other triangles, as many of each).  A
    disk is moved along x; any other picture is cut into upright strips with a
    gap of background, and the strips change places.  All moves are by the
    common period of the lattice and the coarse raster."""
    bm = _picture(w, h, content, torch.Generator(device=_device()).manual_seed(random.Random(key).getrandbits(48)))
    s = _stride(edge)
    period = s
    while period / edge != period // edge:
        period += s
    if content == "disk":
        cols = bm.any(0).nonzero()[:, 0]
        lo, hi = int(cols[0]) // period, (w - 1 - int(cols[-1])) // period
        return bm.roll((seed % (lo + hi + 1) - lo) * period, 1)
    n = max(2, min(8, w // 256))
    width = w // n // period * period
    for j in range(n + 1):
        bm[:, max(0, j * width - int(4 * s + 2 * edge) - 1):j * width] = 0
    # an order other than the neighbouring seeds'
    at, left, order = seed * 7919 % math.factorial(n), list(range(n)), []
    while left:
        order.append(left.pop(at % len(left)))
        at //= len(left) + 1
    return torch.cat([bm[:, j * width:(j + 1) * width] for j in order] + [torch.zeros_like(bm[:, n * width:])], 1)


def _case_bitmap(case, seed):
    return _bitmap(case["w"], case["h"], case["edge"], case["content"], "%(w)d %(h)d %(content)s" % case, seed)


def _requests(case):
    """(width, height, edge, content) of a batch's images: a property of the case."""
    r = random.Random("%(kind)s %(n)d %(lo)d %(hi)d" % case)
    out = []
    for _ in range(case["n"]):
        if case["kind"] == "batch":
            out.append((r.randint(case["lo"], case["hi"]), r.randint(case["lo"], case["hi"]), r.choice((1, 2, 4)),
                        "noise8"))
        else:
            side = _log_int(r, case["lo"], case["hi"])
            out.append((side, side, r.choice((1, 2, 4)), r.choice(("ellipses", "noise8"))))
    return out


def _items(case, seed):
    return [(_bitmap(w, h, float(edge), content, "%s %d" % (content, j), seed + j), float(edge))
            for j, (w, h, edge, content) in enumerate(_requests(case))]


def _outputs(nv: int, nt: int):
    dev = _device()
    return (torch.empty((nv, 2), dtype=torch.float64, device=dev), torch.empty((nt, 3), dtype=torch.int32, device=dev),
            torch.empty((nt,), dtype=torch.uint8, device=dev))


def _pulse(case):
    w, h = case["w"], case["h"]
    return (w - 1) / 2.0, (h - 1) / 2.0, min(w, h) / 8.0


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "batch":
        s["items"] = _items(case, seed)
        b = s["batch"] = Batch(s["items"])
        sizes = b.plan()
        # one arena of each kind for the whole batch, the images' meshes one after the other
        v, t, c = s["out"] = _outputs(sum(z.n_vertices for z in sizes), sum(z.n_triangles for z in sizes))
        views, pv, pt = [], 0, 0
        for z in sizes:
            views.append((v[pv:pv + z.n_vertices], t[pt:pt + z.n_triangles], c[pt:pt + z.n_triangles]))
            pv, pt = pv + z.n_vertices, pt + z.n_triangles
        b.bind(views)
        s["views"] = views
        s["graph"] = b.capture()
        return s
    if kind == "serve":
        s["items"] = _items(case, seed)
        return s
    bm = s["bitmap"] = _case_bitmap(case, seed)
    edge = case["edge"]
    if kind == "mesh":
        s["flags"] = sbmt.BOTH_SIDES if case["both"] else 0
        if case["call"] != "from_bitmap":
            s["ws"] = sbmt.workspace(bm, edge, s["flags"])
            z = sbmt.plan(bm, edge, s["ws"], s["flags"])
            s["out"] = _outputs(z.n_vertices, z.n_triangles)
            s["sizes"] = torch.zeros(5, dtype=torch.int64, device=bm.device)
    elif kind == "grid":
        s["pre"] = Preprocessor(bm, edge)
    elif kind == "alg3":
        if case["call"] == "kept":
            s["pre"] = MeshPreprocessor(bm, edge)
    elif kind == "measure":
        s["verts"], s["tris"], _ = sbmt.mesh_from_bitmap(bm, edge)
        s["field"] = 20.0 + 5.0 * _blur(torch.randn(bm.shape, generator=torch.Generator(device=bm.device).manual_seed(seed),
                                                          device=bm.device), 4.0, 1)
    elif kind == "laplace":
        s["verts"], s["tris"], _ = sbmt.mesh_from_bitmap(bm, edge)
    else:
        m = preprocess_mesh(bm, edge)
        s["verts"], s["tris"] = m.verts, m.tris
        s["lap"] = Laplacian(m.verts, m.tris)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "mesh":
        bm, edge, flags = s["bitmap"], case["edge"], s["flags"]
        if case["call"] == "from_bitmap":
            return sbmt.mesh_from_bitmap(bm, edge, case["both"])
        v, t, c = s["out"]
        if case["call"] == "async":
            sbmt.mesh_async(bm, edge, s["ws"], v, t, c, s["sizes"], flags)
            return v, t, c, s["sizes"]
        z = sbmt.plan(bm, edge, s["ws"], flags)
        sbmt.run(bm, edge, s["ws"], v, t, c, flags)
        return v, t, c, [z.n_vertices, z.n_triangles, z.n_cut, z.n_segments]
    if kind == "batch":
        s["graph"].replay()
        return s["out"]
    if kind == "serve":
        return mesh_batch(s["items"])
    if kind == "grid":
        p = s["pre"]
        n = p.run()
        return p.verts[:n[0]], p.on_polyline[:n[0]], p.tris[:n[1]], list(n)
    if kind == "alg3":
        if case["call"] == "once":
            m = preprocess_mesh(s["bitmap"], case["edge"])
            return m.verts, m.tris, m.codes, [m.n_grid_vertices, m.n_snapped, m.n_repelled, m.n_inserted, m.n_cut]
        p = s["pre"]
        n = p.run()
        return p.verts[:n[0]], p.tris[:n[1]], p.codes[:n[1]], list(n)
    if kind == "measure":
        vv, tv = sample_field(s["field"], s["verts"], s["tris"])
        return vv, tv, mesh_quality(s["verts"], s["tris"])
    if kind == "laplace":
        lap = Laplacian(s["verts"], s["tris"])
        return lap.csr(), lap.info
    lap = s["lap"]
    u = lap.heat_init(*_pulse(case))
    return lap.heat_steps(u, alpha=500.0, dt=1.9 / (500.0 * lap.info["lambda_bound"]), steps=case["steps"])


# -- work ---------------------------------------------------------------------------

def _mesh_counts(w, h, edge, content, both=False):
    """Expected (vertices, triangles) of a mesh: the covered area in base triangles."""
    f = {"disk": math.pi * (20 / 64.0 * min(w, h)) ** 2 / (w * h), "noise8": 0.5, "noise16": 0.382,
         "ellipses": 1.0 - math.exp(-32 * math.pi * 85.0 ** 2 / (w * h))}[content]
    nt = (1.0 if both else f) * w * h / (HALF_SQRT3 / 2 * edge * edge)
    return nt / 2, nt


def work(case):
    kind = case["kind"]
    if kind in ("batch", "serve"):
        byts = flops = 0.0
        for w, h, edge, content in _requests(case):
            nv, nt = _mesh_counts(w, h, edge, content)
            byts += w * h + 16 * nv + 13 * nt
            flops += 4 * nv
        return {"bytes": byts, "flops": flops}
    w, h, edge = case["w"], case["h"], case["edge"]
    nv, nt = _mesh_counts(w, h, edge, case["content"], case.get("both", False))
    nnz = 6 * nv  # neighbours of a vertex, the diagonal not stored
    if kind in ("mesh", "alg3"):  # bitmap in; vertices, triangles, codes out
        return {"bytes": w * h + 16 * nv + 13 * nt, "flops": 4 * nv}
    if kind == "grid":  # bitmap in; every lattice vertex, its byte and two triangles each out
        n = w * h / (HALF_SQRT3 * edge * edge)
        return {"bytes": w * h + 17 * n + 24 * n, "flops": 4 * n}
    if kind == "measure":  # field and mesh in; a value per vertex and triangle out
        return {"bytes": 4 * w * h + 16 * nv + 12 * nt + 8 * nv + 8 * nt, "flops": 15 * nv + 60 * nt}
    if kind == "laplace":  # mesh in; row offsets, columns, weights, masses, boundary bytes out
        return {"bytes": 16 * nv + 12 * nt + 8 * nv + 12 * nnz + 9 * nv, "flops": 40 * nt}
    # the pulse, then per step the operator, masses and boundary read, the field read and written
    return {"bytes": 25 * nv + case["steps"] * (8 * nv + 12 * nnz + 9 * nv + 16 * nv),
            "flops": case["steps"] * (3 * nnz + 4 * nv)}


# -- plain 64-bit results --------------------------------------------------------------

def _exact_vertices(bitmap, edge: float, both: bool):
    """Vertices of the mesh in owner order: every lattice vertex (row, then
    column) gives itself when inside, the crossings of the boundary with its
    edges to (k, i+1), (k+1, i+o-1), (k+1, i+o) in order from it, then the
    boundary point inside its triangle below and inside its triangle to the
    right."""
    dev, f8 = bitmap.device, torch.float64
    H, W = bitmap.shape
    s = _stride(edge)
    ch, cw = -(-H // s), -(-W // s)
    full = torch.zeros((ch * s, cw * s), dtype=torch.uint8, device=dev)
    full[:H, :W] = bitmap != 0
    coarse = 2 * full.view(ch, s, cw, s).sum((1, 3), dtype=torch.int32) >= s * s
    ring = 4
    smp = torch.nn.functional.pad(coarse.to(torch.int64), (ring, ring + 4, ring, ring + 4))
    unit = 1
    while edge * unit != int(edge * unit):
        unit *= 2
    x0 = -(2 * edge + 3) / 4 - (0.0 if unit == 1 else 0.25 / unit)
    nk = 1
    while 3 * (nk * edge) ** 2 <= (2 * s * ch + 1) ** 2:
        nk += 1
    nk += 1
    ni = int((s * cw - 0.5 - x0) // edge) + 2
    off = (s - 1) / 2.0  # the first sample's centre
    out = []
    rows = max(1, (1 << 21) // ni)
    for k0 in range(0, nk, rows):
        k = torch.arange(k0, min(k0 + rows, nk), device=dev)[:, None]
        i = torch.arange(ni, device=dev)[None, :]
        o = k % 2
        y = (-1.0 + (edge * k.to(f8)) * HALF_SQRT3).expand(-1, ni).reshape(-1)
        y1 = (-1.0 + (edge * (k + 1).to(f8)) * HALF_SQRT3).expand(-1, ni).reshape(-1)
        x = (x0 + edge * i.to(f8) + 0.5 * edge * o.to(f8)).reshape(-1)
        r, c = ((y - off) / s).floor().long() + ring, ((x - 0.5 * edge - off) / s).floor().long() + ring
        win = sum(smp[r + a, c + b] for a in range(3) for b in range(3))
        m = torch.zeros((x.numel(), 9), dtype=torch.bool, device=dev)
        xy = torch.zeros((x.numel(), 9, 2), dtype=f8, device=dev)
        # the vertex itself: its place in the cell of four samples around it
        cv = ((x - off) / s).floor().long() + ring
        du, dv = (x - off) / s + ring - cv, (y - off) / s + ring - r
        q = [smp[r, cv], smp[r, cv + 1], smp[r + 1, cv + 1], smp[r + 1, cv]]
        near = [du + dv < 0.5, 1 - du + dv < 0.5, 2 - du - dv < 0.5, du + 1 - dv < 0.5]
        n = sum(q)
        alone = sum(a * b for a, b in zip(q, near)) > 0          # one foreground corner: inside its triangle
        cut = sum((1 - a) * b for a, b in zip(q, near)) > 0      # background corners are cut off
        straight = torch.where(q[0] == q[1], torch.where(dv < 0.5, q[0], q[3]), torch.where(du < 0.5, q[0], q[1]))
        inside = torch.where(n == 4, True, torch.where(n == 0, False, torch.where(n == 1, alone, ~cut)))
        inside = torch.where((n == 2) & (q[0] != q[2]), straight > 0, inside)
        m[:, 0] = True if both else inside
        xy[:, 0, 0], xy[:, 0, 1] = x, y
        # the boundary around the owners whose nine samples differ
        w = ((win != 0) & (win != 9)).nonzero()[:, 0]
        if w.numel():
            mw, xyw = _exact_cuts(smp, r[w], c[w], x[w], y[w], y1[w], edge, s, off, ring)
            m[w, 1:] = mw
            xy[w, 1:] = xyw
        out.append(xy[m])
    return torch.cat(out)


def _exact_cuts(smp, r, c, x, y, y1, edge, s, off, ring):
    """Crossings of the three owned edges (two slots each, in order) and the
    boundary points inside the two owned triangles, of the owners at (x, y)."""
    f8, n = torch.float64, x.numel()
    seg = []  # (present, px, py, qx, qy) of the marching-squares segments of the 2 x 2 cells
    for cell in range(4):
        rr, cc = r + cell // 2, c + cell % 2
        bx, by = off + s * (cc - ring).to(f8), off + s * (rr - ring).to(f8)
        mid = torch.tensor([[0.5, 0.0], [1.0, 0.5], [0.5, 1.0], [0.0, 0.5]], dtype=f8, device=x.device) * s
        q = [smp[rr, cc], smp[rr, cc + 1], smp[rr + 1, cc + 1], smp[rr + 1, cc]]
        # a segment leaves the midpoint where the samples turn from foreground to
        # background (in positive order) and ends at the next turn back
        for a in range(4):
            leave = (q[a] == 1) & (q[(a + 1) % 4] == 0)
            end = torch.full_like(rr, (a + 3) % 4)
            for d in (2, 1):
                e = (a + d) % 4
                end = torch.where((q[e] == 0) & (q[(e + 1) % 4] == 1), e, end)
            seg.append((leave, bx + mid[a, 0], by + mid[a, 1], bx + mid[end, 0], by + mid[end, 1]))
    vx, vy = (x + edge, x - 0.5 * edge, x + 0.5 * edge), (y, y1, y1)
    m = torch.zeros((n, 8), dtype=torch.bool, device=x.device)
    xy = torch.zeros((n, 8, 2), dtype=f8, device=x.device)
    for e in range(3):
        gx, gy = vx[e] - x, vy[e] - y
        pos, pts = [], []
        for ok, px, py, qx, qy in seg:
            dp, dq = gx * (py - y) - gy * (px - x), gx * (qy - y) - gy * (qx - x)
            lu = (qx - px) * (y - py) - (qy - py) * (x - px)
            lv = (qx - px) * (vy[e] - py) - (qy - py) * (vx[e] - px)
            hit = ok & ((dp > 0) != (dq > 0)) & ((lu > 0) != (lv > 0))
            t = dp / torch.where(hit, dp - dq, 1.0)
            pts.append(torch.stack((px + t * (qx - px), py + t * (qy - py)), 1))
            pos.append(torch.where(hit, lu / torch.where(hit, lu - lv, 1.0), math.inf))
        pos, at = torch.stack(pos, 1).sort(1)
        pts = torch.stack(pts, 1)
        for j in range(2):
            m[:, 2 * e + j] = pos[:, j] < math.inf
            xy[:, 2 * e + j] = pts.gather(1, at[:, j, None, None].expand(-1, 1, 2))[:, 0]
    tri = (((x, y), (vx[2], y1), (vx[1], y1)), ((x, y), (vx[0], y), (vx[2], y1)))
    for t in range(2):
        for ok, px, py, qx, qy in seg:
            hit = ok.clone()
            for a in range(3):
                (ax, ay), (bx, by) = tri[t][a], tri[t][(a + 1) % 3]
                hit &= (bx - ax) * (qy - ay) - (by - ay) * (qx - ax) > 0
            m[:, 6 + t] |= hit
            xy[:, 6 + t] = torch.where(hit[:, None], torch.stack((qx, qy), 1), xy[:, 6 + t])
    return m, xy


def _exact_operator(v, t):
    """Rows of the cotangent Laplacian: neighbours in order of first appearance
    over a vertex's triangles (ascending, next vertex then previous), half
    cotangents summed; lumped masses, boundary flags, the Gershgorin bound."""
    nv, t = v.shape[0], t.long()
    p = v[t]
    e1, e2 = p[:, 1] - p[:, 0], p[:, 2] - p[:, 0]
    cross = e1[:, 0] * e2[:, 1] - e1[:, 1] * e2[:, 0]
    cot = torch.stack([0.5 * (((p[:, (k + 1) % 3] - p[:, k]) * (p[:, (k + 2) % 3] - p[:, k])).sum(1) / cross)
                       for k in range(3)], 1)
    nxt, prv = [1, 2, 0], [2, 0, 1]
    i, order = t.reshape(-1).sort(stable=True)
    j = torch.stack((t[:, nxt].reshape(-1)[order], t[:, prv].reshape(-1)[order]), 1).reshape(-1)
    wt = torch.stack((cot[:, prv].reshape(-1)[order], cot[:, nxt].reshape(-1)[order]), 1).reshape(-1)
    i = i.repeat_interleave(2)
    key, inv, count = torch.unique(i * nv + j, return_inverse=True, return_counts=True)
    first = torch.full_like(key, 1 << 62).scatter_reduce(0, inv, torch.arange(i.numel(), device=v.device), "amin")
    val = torch.zeros(key.numel(), dtype=torch.float64, device=v.device).index_add(0, inv, wt)
    order = first.argsort()
    row, val, once = key[order] // nv, val[order], count[order] == 1
    zero = torch.zeros(nv, dtype=torch.float64, device=v.device)
    mass = zero.index_add(0, t.reshape(-1), (0.5 * cross / 3.0).repeat_interleave(3))
    bound = (zero.index_add(0, row, val) + zero.index_add(0, row, val.abs())) / mass
    bnd = torch.zeros(nv, dtype=torch.bool, device=v.device)
    bnd[row[once]] = True
    return {"row": row, "col": key[order] % nv, "val": val, "mass": mass, "boundary": bnd, "lambda": float(bound.max())}


def _exact_sample(field, v, t):
    f = field.double()
    H, W = f.shape
    x, y = v[:, 0].clamp(0, W - 1), v[:, 1].clamp(0, H - 1)
    c0, r0 = x.long(), y.long()
    c1, r1 = (c0 + 1).clamp(max=W - 1), (r0 + 1).clamp(max=H - 1)
    a, b = x - c0, y - r0
    val = (1 - a) * (1 - b) * f[r0, c0] + a * (1 - b) * f[r0, c1] + (1 - a) * b * f[r1, c0] + a * b * f[r1, c1]
    return val, val[t.long()].sum(1) / 3.0


def _exact_quality(v, t):
    p = v[t.long()]
    e = torch.stack([p[:, (k + 1) % 3] - p[:, k] for k in range(3)], 1)
    len2 = (e * e).sum(2)
    cross = e[:, 0, 0] * (p[:, 2, 1] - p[:, 0, 1]) - e[:, 0, 1] * (p[:, 2, 0] - p[:, 0, 0])
    ar = (len2.amax(1) / cross.abs()).sort().values
    area, n = 0.5 * cross, cross.numel()
    j = len2.argmin(1)
    prod = len2.prod(1) / len2.gather(1, j[:, None])[:, 0]
    k = int((cross * cross / prod).argmin())
    apex = (int(j[k]) + 2) % 3
    a, b = p[k, (apex + 1) % 3] - p[k, apex], p[k, (apex + 2) % 3] - p[k, apex]
    angle = math.degrees(math.atan2(abs(float(a[0] * b[1] - a[1] * b[0])), float((a * b).sum())))
    whole = ("n_triangles", "n_invalid", "n_nonpositive", "n_slivers", "n_equilateral", "min_angle_tri", "angle_hist")
    return dict({w: None for w in whole}, min_angle_deg=angle, min_area=float(area.min()), max_area=float(area.max()),
                mean_area=float(area.mean()), var_area=float(area.var(correction=0)),
                ar_median=float(ar[(n + 1) // 2 - 1]), ar_p95=float(ar[(95 * n + 99) // 100 - 1]), ar_max=float(ar[-1]))


def exact(case, seed):
    kind = case["kind"]
    if kind == "mesh":
        v = _exact_vertices(_case_bitmap(case, seed), case["edge"], case["both"])
        return (v, None, None) + ((None,) if case["call"] != "from_bitmap" else ())
    if kind == "batch":
        return torch.cat([_exact_vertices(b, e, False) for b, e in _items(case, seed)]), None, None
    if kind == "serve":
        return [(_exact_vertices(b, e, False), None, None) for b, e in _items(case, seed)]
    if kind in ("grid", "alg3"):
        return None  # moved vertices: held to the bound of their type
    s = prepare(case, seed)  # the mesh is an input here
    if kind == "measure":
        return _exact_sample(s["field"], s["verts"], s["tris"]) + (_exact_quality(s["verts"], s["tris"]),)
    op = _exact_operator(s["verts"], s["tris"])
    if kind == "laplace":
        csr = {"row_off": None, "col": None, "val": op["val"], "mass": op["mass"], "boundary": None}
        return csr, {"min_mass": float(op["mass"].min()), "lambda_bound": op["lambda"], "n_vertices": None, "nnz": None,
                     "n_boundary": None, "n_invalid": None}
    x0, y0, sigma = _pulse(case)
    d = s["verts"] - torch.tensor([x0, y0], dtype=torch.float64, device=s["verts"].device)
    u = torch.where(op["boundary"], 0.0, 100.0 * torch.exp(-(d * d).sum(1) / (2.0 * sigma * sigma)))
    dt = 1.9 / (500.0 * op["lambda"])
    for _ in range(case["steps"]):
        ku = torch.zeros_like(u).index_add(0, op["row"], op["val"] * (u[op["row"]] - u[op["col"]]))
        u = torch.where(op["boundary"], 0.0, u - dt * 500.0 * ku / op["mass"])
    return u
