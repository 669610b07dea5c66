// sbmt_pre.h -- geometric preprocessing of Alg. 3 (Sec. 3.5) and the
// retriangulation of the preprocessed grid: device code and workspace layout.
// Included by sbmt.hip inside namespace sbmt, after the meshing kernels whose
// helpers it uses (raster layout, row segments, scans).
#pragma once

// ---------------------------------------------------------------------------
// Geometric preprocessing of Alg. 3 (Sec. 3.5, thresholds of Sec. 3.3.4):
// Step 1 snaps a lattice vertex to the polyline vertex within distance a,
// Step 2 moves a vertex within c of a segment along that segment's normal to
// distance exactly c, Step 3 splits every mesh edge within b of a polyline
// vertex that no lattice vertex snapped to, at that vertex (the edge's one or
// two triangles become a fan around it).  The result is the preprocessed
// grid: lattice vertices (moved), inserted polyline vertices, and the base
// triangles with their split edges fanned.
//
// Polyline vertices are the marching-squares midpoints whose two coarse
// samples differ; distances are square roots of sums of squares in double
// precision, evaluated exactly as written (no contraction).  Admissible
// thresholds (b < a/2, c < a/sqrt2, a < h/2) keep every decision local: at
// most one polyline vertex within a of a lattice vertex, at most one segment
// within c of an unsnapped one, at most one edge within b of a polyline vertex
// and at most one polyline vertex within b of an edge, at most one split edge
// per triangle; the kernels flag a protocol error otherwise.
// ---------------------------------------------------------------------------
// A cut grid triangle's output.  Its points are numbered 0..2 the corners, 3..6
// the ends of its one or two pieces that are crossings of its edges, 7 the
// polyline vertex inside.
// At most four output triangles: it holds two segments at most, so either up to four
// crossings lie on its boundary (seven points there with the corners: five triangles
// on both sides of the polyline together) or two and a vertex inside (five points and
// one inside: five triangles), and one at least is background.
constexpr int kPreKeep = 4;
struct PreCut {
  uint32_t head;      // bits 0..7 triangles; 8 + 4 e: edge slot of edge e at its owner
  uint32_t ends;      // end k at bits 8 k: edge (bits 0, 1), order along the edge from its lower-numbered corner (2, 3),
                      // 7: it is a crossing
  uint32_t tri[2];    // two triangles each, 9 bits a triangle: three points of three bits
  int32_t id[3];      // corners
  int32_t eo[3];      // owner of edge e (corner e to e + 1)
  int32_t pad[2];
  double2 pos[5];     // the crossings' and the inner vertex's places
};
static_assert(sizeof(PreCut) == 128, "one line");
// 64 grid vertices: which of them the mesh uses, and the used ones before them
// in their block of kPreVScan.
struct PreUsed {
  uint64_t bits;
  int32_t base, pad;
};

constexpr int kPreStamp = 6;  // words
struct PreArgs {
  double a, b, c;
  double* verts;         // [NK NI + inserted][2]: lattice vertex k NI + i first (the mesh: moved and inserted ones only)
  uint8_t* on_polyline;  // per vertex: sits on a polyline vertex (null: not asked for)
  int32_t* tris;         // [triangles][3]
  int64_t vcap, tcap;
  int wshift;            // log2 of the raster words a wave enumerates the polyline from (pre_wave_words)
  uint8_t* mid;          // per midpoint: 1 if a lattice vertex snapped to it
  uint8_t* flags;        // per lattice vertex: bits 0-2 owned side E0-E2 split, 3 moved, 4 claimed, 5 snapped
  int32_t* split;        // [NK NI][3]: midpoint splitting side E0, E1, E2 (written where split)
  int64_t* ins_base;     // [NK NI]: first inserted vertex of the owner (written where it has one)
  int64_t* counts;       // [8 + 512]: [2] error, [3] touched owners, [4] cut triangles (mesh); from kPreTally 256 counters of snapped, then of repelled vertices
  uint32_t* touched;     // [NK][8 NCB]: bit per owner, those a segment can reach (mesh)
  int64_t ntouched;      // its words
  int32_t* snap_mid;     // [NK NI]: the polyline vertex a lattice vertex snapped to (written where snapped)
  // retriangulation of the grid (sbmt_preprocess_mesh)
  uint64_t* inside;      // [4 segments]: bit per owner, the untouched ones inside (their slots are kept whole)
  uint32_t* rcount;      // [NK NI]: per-owner counts (pre_rc_*), of the touched owners
  uint32_t* rtri;        // [NK NI], of the touched owners: per grid triangle of the owner (4): output triangles (6 bits each), inner-vertex bits 24..27, cut bits 28..31
  int64_t* rbase;        // [NK NI]: first new vertex of the owner (written where it has one)
  const int64_t* gsizes; // the grid phase's sizes record (grid vertices first)
  int32_t* otris;        // [otcap][3]
  uint8_t* ocodes;       // [otcap]
  int64_t otcap;
  // compaction of the mesh's vertices: the grid vertices some output triangle
  // uses (marked in the count pass) keep their order and come first
  double* overts;        // [ovcap][2]: the mesh's vertices
  int64_t ovcap;
  uint8_t* used;         // [usedcap]: grid vertex used by an output triangle
  int64_t usedcap;
  PreUsed* uword;        // [usedcap / 64]: the same as bits, with their ranks
  int32_t* tlist;        // [NK NI]: the touched owners, in owner order
  int64_t* rtbase;       // [NK NI]: a touched owner's first output triangle
  int64_t* vbsum;        // per block of kPreVScan grid vertices: used count, then base
  int64_t* nused;        // [1]: grid vertices in the mesh
  // the cut grid triangles, numbered (slots)
  int32_t* cbase;        // [NK NI]: first slot of list position t
  uint64_t* citem;       // [ccap]: list position * 4 + grid triangle of each slot
  PreCut* cstore;        // [ccap]: its output, kept by the count pass for the triangle pass
  int64_t ccap;
  // the workspace's stamp: what a finished plan leaves there, and what this call's image and thresholds make it
  uint64_t* stamp_at;
  uint64_t stamp[kPreStamp];
};
constexpr int kPreVScan = 16384;  // grid vertices per block of the compaction scan
constexpr int kPreApplyWords = 16;  // words of 64 grid vertices per block that copies the used ones
static_assert(kPreVScan % (64 * kPreApplyWords) == 0, "in one block of the scan");
// Whether the workspace holds the plan of this image size, edge and thresholds.
// The passes that write the mesh follow indices and bounds from the workspace, so
// each looks at this first: they must not run after a plan that failed, over
// another image's, or over memory that was never planned.  The stamp is in words
// that every call's k_coarsen clears, and the last pass of a plan without an error
// sets it.  The passes take a count or a bound of 0 without it rather than
// return, so that its load and the first ones of the pass wait together.
__device__ __forceinline__ bool pre_planned(const PreArgs& P) {
  uint64_t d = 0;
#pragma unroll
  for (int q = 0; q < kPreStamp; ++q) d |= P.stamp_at[q] ^ P.stamp[q];
  return d == 0;
}
constexpr uint8_t kPreMoved = 8;
constexpr int kPreTally = 8;
constexpr int kPreCounts = kPreTally + 512;

// Midpoint ids: horizontal midpoint between samples (R, C) and (R, C+1) is
// 2 ((R + 1)(CW + 2) + C + 1), the vertical one between (R, C) and (R+1, C)
// one more; R in -1 .. CH, C in -1 .. CW.
__device__ __forceinline__ int64_t mid_id(const Geo& g, int R, int C, int vert) {
  return 2 * ((int64_t)(R + 1) * (g.CW + 2) + (C + 1)) + vert;
}
__device__ __forceinline__ int sample_at(const Img& d, const Geo& g, int R, int C) {
  if (R < 0 || R >= g.CH || C < 0 || C >= g.CW) return 0;
  const int rr = R + kRing, cc = C + kRingC;
  return (int)((d.bits[(int64_t)rr * g.wpr + (cc >> 5)] >> (cc & 31)) & 1u);
}
// Sample (R, C) sits at pixel (s C + (s-1)/2, s R + (s-1)/2); the offset:
__device__ __forceinline__ double sample_off(const Geo& g) { return 0.5 * (g.s - 1); }
__device__ __forceinline__ double euclid_d(double dx, double dy) { return __builtin_sqrt(dx * dx + dy * dy); }
// distance from (x, y) to segment P -> Q and the parameter of the closest point
__device__ __forceinline__ double seg_dist_d(double x, double y, double px, double py, double qx, double qy, double* tp) {
  const double dx = qx - px, dy = qy - py;
  double t = ((x - px) * dx + (y - py) * dy) / (dx * dx + dy * dy);
  t = t < 0.0 ? 0.0 : (t > 1.0 ? 1.0 : t);
  if (tp) *tp = t;
  return euclid_d(x - (px + t * dx), y - (py + t * dy));
}
__device__ __forceinline__ int floor_index(const Geo& g, double v) {
  return (int)__builtin_floor((v - sample_off(g)) / g.s);
}

// thresholds widened by a relative and absolute margin far above the rounding
// of the box bounds, so that a box never misses a candidate; the distances to a
// line that decide early are held to it, too (the distance that decides carries
// the rounding of whole coordinates, 1e-12 px at 8192 px, whatever the threshold)
__device__ __forceinline__ double widen(double r) { return r * (1.0 + 1e-12) + 1e-9; }
// Segment j of marching-squares case cs of dual cell (R, C): end points in pixels.
__device__ __forceinline__ void cell_segment(const Geo& g, int R, int C, uint32_t ms, int j, double& px, double& py,
                                             double& qx, double& qy) {
  const int ea = (int)((ms >> (2 + 4 * j)) & 3u), eb = (int)((ms >> (4 + 4 * j)) & 3u);
  // cell edges: 0 top, 1 right, 2 bottom, 3 left (midpoints relative to the TL sample, in s/2)
  const double x0 = (double)g.s * C + sample_off(g), y0 = (double)g.s * R + sample_off(g), hs = 0.5 * g.s;
  px = x0 + (ea == 0 || ea == 2 ? hs : (ea == 1 ? 2.0 * hs : 0.0));
  py = y0 + (ea == 1 || ea == 3 ? hs : (ea == 2 ? 2.0 * hs : 0.0));
  qx = x0 + (eb == 0 || eb == 2 ? hs : (eb == 1 ? 2.0 * hs : 0.0));
  qy = y0 + (eb == 1 || eb == 3 ? hs : (eb == 2 ? 2.0 * hs : 0.0));
}

// Base triangle slot t of owner (k, i) exists (all three corners in the lattice).
__device__ __forceinline__ bool pre_slot_ok(const Geo& g, int k, int i, int t) {
  const int o = k & 1;
  return t == 0 ? (k + 1 < g.NK && i + o - 1 >= 0 && i + o < g.NI) : (k + 1 < g.NK && i + 1 < g.NI && i + o < g.NI);
}
// Owned side e of (k, i) is a side of some base triangle: E0 of Ta(k, i) or of
// Tb of the owner above whose lower side it is, E1 of Tb(k, i) or of
// Ta(k, i-1), E2 of either triangle of (k, i).
__device__ __forceinline__ bool pre_edge_live(const Geo& g, int k, int i, int e) {
  if (e == 0) {
    const int ia = i + 1 - ((k - 1) & 1);
    return pre_slot_ok(g, k, i, 1) || (k >= 1 && ia >= 0 && ia < g.NI && pre_slot_ok(g, k - 1, ia, 0));
  }
  if (e == 1) return pre_slot_ok(g, k, i, 0) || (i >= 1 && pre_slot_ok(g, k, i - 1, 1));
  return pre_slot_ok(g, k, i, 0) || pre_slot_ok(g, k, i, 1);
}

// Flag bits per lattice vertex: 0-2 owned side E0-E2 split, 3 moved, 4 taken
// by a segment (Step 2), 5 snapped (Step 1).
constexpr uint32_t kPreClaim = 16;
constexpr uint32_t kPreSnapped = 32;
// ORs bits into the flag byte of vertex v; returns the byte before.
__device__ __forceinline__ uint32_t pre_flag_or(uint8_t* flags, int64_t v, uint32_t bits) {
  const int sh = 8 * (int)(v & 3);
  const uint32_t old = atomicOr(reinterpret_cast<uint32_t*>(flags + (v & ~(int64_t)3)), bits << sh);
  return (old >> sh) & 0xffu;
}
__device__ __forceinline__ void pre_error(const PreArgs& P) { atomicOr((unsigned long long*)&P.counts[2], 1ull); }
// Wave sum of n added to one of 256 counters of tally `which` (0 snapped,
// 1 repelled); every lane of the wave must call it.
__device__ __forceinline__ void pre_tally(const PreArgs& P, int which, int n) {
  const int tot = __builtin_amdgcn_readlane(wave_incl_scan_dpp(n), 63);
  if ((threadIdx.x & 63) == 0 && tot) {
    const int slot = (int)((blockIdx.x * 4u + (threadIdx.x >> 6)) & 255u);
    atomicAdd((unsigned long long*)&P.counts[kPreTally + 256 * which + slot], (unsigned long long)tot);
  }
}
// Lattice column pitch and row spacing in pixels (to locate rows and columns;
// positions themselves always come from lat_x / lat_y).
__device__ __forceinline__ double pre_hx(const Geo& g) { return (double)g.h / g.U; }
__device__ __forceinline__ double pre_hy(const Geo& g) { return pre_hx(g) * kHalfSqrt3; }
__device__ __forceinline__ int pre_row_floor(const Geo& g, double y) { return (int)__builtin_floor((y + 1.0) / pre_hy(g)); }
__device__ __forceinline__ int pre_lat_X(const Geo& g, int k, int i) { return g.X0 + 4 * g.h * i + 2 * g.h * (k & 1); }
// Owner column of x in row k, as a real number (column i sits at z = i).
__device__ __forceinline__ double pre_col(const Geo& g, int k, double x) {
  return (x - lat_x(g, pre_lat_X(g, k, 0))) / pre_hx(g);
}

// x, y or z for j = 0, 1, 2: selects rather than an indexed local array,
// which would live in scratch memory.
template <class V>
__device__ __forceinline__ V pre_sel3(const V& x, const V& y, const V& z, int j) {
  return j == 0 ? x : (j == 1 ? y : z);
}
// Place of lattice vertex v = (k, i) with flags f: the grid stores everyone's
// (kAll), the mesh only the moved ones' (1.2 GB less to write and read back on
// 8192 x 8192).  A select and no branch, so that the loads of a triangle's corners
// are in flight together (k_pre_count, its check still on the waves as they fell,
// with branches 563 us, so 437; with every place stored 344).
template <bool kAll>
__device__ __forceinline__ double2 pre_place(const PreArgs& P, const Geo& g, int64_t v, int k, int i, uint32_t f) {
  const double2* const V = reinterpret_cast<const double2*>(P.verts);
  if (kAll) return V[v];
  const bool moved = (f & kPreMoved) != 0;
  const double2 m = V[moved ? v : 0];
  const double x = lat_x(g, pre_lat_X(g, k, i)), y = lat_y(g, k);
  return make_double2(moved ? m.x : x, moved ? m.y : y);
}
// The unmoved lattice: every vertex at its lattice position.
// Block: 1024 vertices of one row, four per thread (stride 256).
constexpr int kPreQuad = 4 * kCB;
__global__ void __launch_bounds__(256) k_pre_lattice(OneSrc src, PreArgs P, int nchunk) {
  const Geo g = src.d.g;
  const int k = (int)(blockIdx.x / (unsigned)nchunk);
  const int i0 = (int)(blockIdx.x - (unsigned)k * (unsigned)nchunk) * kPreQuad + (int)threadIdx.x;
  const double y = lat_y(g, k);
  double2* V = reinterpret_cast<double2*>(P.verts);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int i = i0 + j * kCB;
    if (i >= g.NI) break;
    const int64_t v = (int64_t)k * g.NI + i;
    if (v < P.vcap) {
      V[v] = make_double2(lat_x(g, pre_lat_X(g, k, i)), y);
      P.on_polyline[v] = 0;
    }
  }
}

// The polyline is enumerated from the coarse raster, stored words of coarse rows
// -1 .. CH - 1: a wave takes 2^wshift of them, one a lane.  Bit j concerns column
// C = C0 + j: dh marks the horizontal midpoint (R, C)-(R, C+1) as a polyline
// vertex, dv the vertical one (R, C)-(R+1, C), and cur / c1 / bel / b1 hold
// the samples (R, C), (R, C+1), (R+1, C), (R+1, C+1) of dual cell (R, C).
struct PreWord {
  int R, C0;
  uint32_t cur, c1, bel, b1, dh, dv;
};
__device__ __forceinline__ void pre_word_at(const Geo& g, uint32_t t, int& R, int& C0) {
  const uint32_t r = t / (uint32_t)g.wpr;
  R = (int)r - 1;
  C0 = 32 * (int)(t - r * (uint32_t)g.wpr) - kRingC;
}
__device__ __forceinline__ uint32_t pre_wave_word0(const PreArgs& P) { return (blockIdx.x * 4u + (threadIdx.x >> 6)) << P.wshift; }
__device__ __forceinline__ bool pre_word(const Img& d, const Geo& g, const PreArgs& P, PreWord& W) {
  const uint32_t lane = threadIdx.x & 63u, t = pre_wave_word0(P) + lane;
  if (lane >> P.wshift || t >= (uint32_t)((g.CH + 1) * g.wpr)) return false;
  pre_word_at(g, t, W.R, W.C0);
  const int w = (W.C0 + kRingC) >> 5;
  const uint32_t* row = d.bits + (int64_t)(W.R + kRing) * g.wpr;
  const bool more = w + 1 < g.wpr;
  W.cur = row[w];
  W.bel = row[g.wpr + w];
  W.c1 = (W.cur >> 1) | ((more ? row[w + 1] : 0u) << 31);
  W.b1 = (W.bel >> 1) | ((more ? row[g.wpr + w + 1] : 0u) << 31);
  W.dh = W.cur ^ W.c1;
  W.dv = W.cur ^ W.bel;
  return true;
}
__device__ __forceinline__ void pre_mid_xy(const Geo& g, int R, int C, int vt, double& x, double& y) {
  x = (double)g.s * C + sample_off(g) + (vt ? 0.0 : 0.5 * g.s);
  y = (double)g.s * R + sample_off(g) + (vt ? 0.5 * g.s : 0.0);
}
// The items the lanes of a wave found (set bits of m0, then of m1; each with a
// 4-bit payload per bit read from pay0 / pay1 when given) are gathered in LDS,
// those that keep(source lane, which mask, bit) refuses dropped when given, and
// dealt round-robin to the lanes: f(source lane, which mask, bit, payload).
// Every thread of the block must call it (it synchronises the block).
constexpr int kPreDeal = 64 * 64;
struct PreKeepAll {
  static constexpr bool all = true;
  __device__ __forceinline__ bool operator()(int, int, int) const { return true; }
};
template <class F>
struct PreKeepIf {
  static constexpr bool all = false;
  F f;
  __device__ __forceinline__ bool operator()(int sl, int which, int bit) const { return f(sl, which, bit); }
};
template <class Pay, class F, class Keep = PreKeepAll>
__device__ __forceinline__ void pre_deal(uint16_t (*lds)[kPreDeal], uint32_t m0, uint32_t m1, Pay pay, F f,
                                         Keep keep = Keep()) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int n = __builtin_popcount(m0) + __builtin_popcount(m1);
  const int incl = wave_incl_scan_dpp(n);
  int total = __builtin_amdgcn_readlane(incl, 63);
  int pos = incl - n;
  for (int which = 0; which < 2; ++which) {
    uint32_t m = which ? m1 : m0;
    while (m) {
      const int j = __builtin_ctz(m);
      m &= m - 1u;
      lds[wv][pos++] = (uint16_t)(lane | (which << 6) | (j << 7) | (pay(which, j) << 12));
    }
  }
  __syncthreads();
  if constexpr (!Keep::all) {
    // the kept ones to the front, in place (a write stays behind the reads)
    int kept = 0;
    for (int q = 0; q < total; q += 64) {  // uniform per wave
      const uint32_t e = q + lane < total ? lds[wv][q + lane] : 0u;
      const bool k = q + lane < total && keep((int)(e & 63u), (int)((e >> 6) & 1u), (int)((e >> 7) & 31u));
      const unsigned long long bal = __ballot(k);
      if (k) lds[wv][kept + lanes_below(bal)] = (uint16_t)e;
      kept += (int)__popcll(bal);
    }
    total = kept;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  for (int q = lane; q < total; q += 64) {
    const uint32_t e = lds[wv][q];
    f((int)(e & 63u), (int)((e >> 6) & 1u), (int)((e >> 7) & 31u), e >> 12);
  }
}
__device__ __forceinline__ uint32_t pre_no_pay(int, int) { return 0u; }

// Step 1 from the polyline side: the lattice vertex within a of polyline vertex
// (R, C, vt) at (mx, my) is the nearest one of a row within a of my (a < h/2:
// lattice vertices are h apart, so there is at most one); it moves onto the
// polyline vertex.  Returns the number of vertices snapped.
__device__ int pre_snap_one(const PreArgs& P, const Geo& g, int R, int C, int vt) {
  double mx, my;
  pre_mid_xy(g, R, C, vt, mx, my);
  const double aw = widen(P.a);
  int hits = 0;
  for (int k = max(0, pre_row_floor(g, my - aw)); k <= min(g.NK - 1, pre_row_floor(g, my + aw)); ++k) {
    const double yv = lat_y(g, k);
    if (!(__builtin_fabs(yv - my) <= aw)) continue;
    const int i = (int)__builtin_floor(pre_col(g, k, mx) + 0.5);
    if (i < 0 || i >= g.NI) continue;
    const double xv = lat_x(g, pre_lat_X(g, k, i));
    if (!(euclid_d(xv - mx, yv - my) < P.a)) continue;
    ++hits;
    const int64_t v = (int64_t)k * g.NI + i;
    if (pre_flag_or(P.flags, v, kPreSnapped | kPreMoved) & kPreSnapped) pre_error(P);  // two polyline vertices
    if (v < P.vcap) {
      reinterpret_cast<double2*>(P.verts)[v] = make_double2(mx, my);
      if (P.on_polyline) P.on_polyline[v] = 1;
    }
    P.mid[mid_id(g, R, C, vt)] = 1;
    P.snap_mid[v] = (int32_t)mid_id(g, R, C, vt);
  }
  if (hits > 1) pre_error(P);
  return hits;
}
__global__ void __launch_bounds__(256) k_pre_snap(OneSrc src, PreArgs P) {
  __shared__ uint16_t lds[4][kPreDeal];
  const Img& d = src.d;
  const Geo g = d.g;
  PreWord W;
  const bool on = P.a > 0.0 && pre_word(d, g, P, W);
  int n = 0;
  const uint32_t base = pre_wave_word0(P);
  pre_deal(lds, on ? W.dh : 0u, on ? W.dv : 0u, pre_no_pay, [&](int sl, int vt, int j, uint32_t) {
    int R, C0;
    pre_word_at(g, base + sl, R, C0);
    n += pre_snap_one(P, g, R, C0 + j, vt);
  });
  pre_tally(P, 0, n);
}

// Step 2 from the segment side: every lattice vertex not snapped within c of
// segment P -> Q moves along the segment's left normal to distance c on its
// own side.  A vertex taken by two segments, or whose closest point is an end
// of the segment, is a protocol error (c < a/sqrt2 excludes both).  Returns
// the number of vertices moved.
__device__ int pre_repel_seg(const PreArgs& P, const Geo& g, double px, double py, double qx, double qy) {
  const double cw = widen(P.c);
  const double x0 = __builtin_fmin(px, qx) - cw, x1 = __builtin_fmax(px, qx) + cw;
  const double y0 = __builtin_fmin(py, qy) - cw, y1 = __builtin_fmax(py, qy) + cw;
  int n = 0;
  const double ex = qx - px, ey = qy - py, reach = cw * cw * (ex * ex + ey * ey);
  for (int k = max(0, pre_row_floor(g, y0)); k <= min(g.NK - 1, pre_row_floor(g, y1)); ++k) {
    const double yv = lat_y(g, k);
    if (yv < y0 || yv > y1) continue;
    const int i0 = max(0, (int)__builtin_floor(pre_col(g, k, x0))), i1 = min(g.NI - 1, (int)__builtin_floor(pre_col(g, k, x1)));
    for (int i = i0; i <= i1; ++i) {
      const double xv = lat_x(g, pre_lat_X(g, k, i));
      if (xv < x0 || xv > x1) continue;
      const double off = ex * (yv - py) - ey * (xv - px);
      if (off * off > reach) continue;  // farther from the line than c, by more than rounding
      const int64_t v = (int64_t)k * g.NI + i;
      if (P.flags[v] & kPreSnapped) continue;
      double t;
      if (!(seg_dist_d(xv, yv, px, py, qx, qy, &t) < P.c)) continue;
      if (pre_flag_or(P.flags, v, kPreClaim | kPreMoved) & kPreClaim) pre_error(P);
      if (!(t > 0.0 && t < 1.0)) pre_error(P);
      const double dx = qx - px, dy = qy - py, L = euclid_d(dx, dy);
      const double nx = -dy / L, ny = dx / L;             // left normal
      const double ds = (xv - px) * nx + (yv - py) * ny;  // signed distance to the line
      const double move = (ds > 0 ? P.c : -P.c) - ds;
      if (v < P.vcap) reinterpret_cast<double2*>(P.verts)[v] = make_double2(xv + move * nx, yv + move * ny);
      ++n;
    }
  }
  return n;
}
__global__ void __launch_bounds__(256) k_pre_repel(OneSrc src, PreArgs P) {
  __shared__ uint16_t lds[4][kPreDeal];
  const Img& d = src.d;
  const Geo g = d.g;
  PreWord W;
  const bool on = P.c > 0.0 && pre_word(d, g, P, W);
  const uint32_t cells = on ? (W.dh | W.dv | (W.cur ^ W.b1)) : 0u;  // dual cells whose samples differ
  int n = 0;
  const uint32_t base = pre_wave_word0(P);
  auto cs_of = [&](int, int j) {
    return ((W.cur >> j) & 1u) | (((W.c1 >> j) & 1u) << 1) | (((W.b1 >> j) & 1u) << 2) | (((W.bel >> j) & 1u) << 3);
  };
  pre_deal(lds, cells, 0u, cs_of, [&](int sl, int, int j, uint32_t cs) {
    int R, C0;
    pre_word_at(g, base + sl, R, C0);
    const uint32_t ms = ms_case((int)cs);
    for (int q = 0; q < (int)(ms & 3u); ++q) {
      double px, py, qx, qy;
      cell_segment(g, R, C0 + j, ms, q, px, py, qx, qy);
      n += pre_repel_seg(P, g, px, py, qx, qy);
    }
  });
  pre_tally(P, 1, n);
}

// Step 3 from the polyline side: a free polyline vertex (no lattice vertex
// snapped to it) finds the base triangle sides within b of it, on the moved
// vertices.  The vertices moved by less than a, so such a side lies within
// r = a + b of the polyline vertex on the lattice: per row, the owners whose
// side e spans x within r (E0 of rows within r of y, E1 and E2 of rows whose
// band reaches y within r).  One side: it is split there (its owner's flag
// bit and split record); more than one, or a side split twice, is a protocol
// error (b < a/2 excludes both).
template <bool kAll>
__device__ void pre_split_one(const PreArgs& P, const Geo& g, int64_t id, double mx, double my) {
  const double r = widen(P.a + P.b), rr = r / pre_hx(g), bw = widen(P.b);
  int nh = 0;
  int64_t hv = -1;
  int he = 0;
  for (int k = max(0, pre_row_floor(g, my - r) - 1); k <= min(g.NK - 1, pre_row_floor(g, my + r)); ++k) {
    const double yu = lat_y(g, k), yd = lat_y(g, k + 1), z = pre_col(g, k, mx);
    const int o = k & 1;
    for (int e = 0; e < 3; ++e) {
      const double yw = e == 0 ? yu : yd;
      if (my < yu - r || my > yw + r) continue;
      // side e of owner i spans columns [i, i+1], [i-1/2, i], [i, i+1/2]
      const double lo = e == 0 ? z - 1.0 - rr : (e == 1 ? z - rr : z - 0.5 - rr);
      const double hi = e == 0 ? z + rr : (e == 1 ? z + 0.5 + rr : z + rr);
      const int kw = e == 0 ? k : k + 1;
      for (int i = max(0, (int)__builtin_floor(lo)); i <= min(g.NI - 1, (int)__builtin_floor(hi)); ++i) {
        if (!pre_edge_live(g, k, i, e)) continue;
        const int iw = e == 0 ? i + 1 : (e == 1 ? i + o - 1 : i + o);
        const double xu = lat_x(g, pre_lat_X(g, k, i)), xw = lat_x(g, pre_lat_X(g, kw, iw));
        if (mx < __builtin_fmin(xu, xw) - r || mx > __builtin_fmax(xu, xw) + r) continue;
        const int64_t v = (int64_t)k * g.NI + i;
        const int64_t vw = (int64_t)kw * g.NI + iw;
        const double2 U = pre_place<kAll>(P, g, v, k, i, kAll ? 0u : P.flags[v]),
                      Wv = pre_place<kAll>(P, g, vw, kw, iw, kAll ? 0u : P.flags[vw]);
        const double dx = Wv.x - U.x, dy = Wv.y - U.y, off = dx * (my - U.y) - dy * (mx - U.x);
        if (off * off > bw * bw * (dx * dx + dy * dy)) continue;  // farther from the line than b, by more than rounding
        // both orientations, as the side's two triangles see it
        if (seg_dist_d(mx, my, U.x, U.y, Wv.x, Wv.y, nullptr) < P.b ||
            seg_dist_d(mx, my, Wv.x, Wv.y, U.x, U.y, nullptr) < P.b) {
          ++nh;
          hv = v;
          he = e;
        }
      }
    }
  }
  if (nh > 1) pre_error(P);
  if (nh == 0) return;
  if (pre_flag_or(P.flags, hv, 1u << he) & (1u << he)) pre_error(P);  // a side split twice
  P.split[3 * hv + he] = (int32_t)id;
}
// Two in three polyline vertices have been snapped to: they are dropped before
// the deal, so that the lanes that look for sides are full, and a side's
// distance is taken only where the vertex lies within b of its line (together
// 125 -> 106 us on 4000 x 3000).
template <bool kAll>
__global__ void __launch_bounds__(256) k_pre_split(OneSrc src, PreArgs P) {
  __shared__ uint16_t lds[4][kPreDeal];
  const Img& d = src.d;
  const Geo g = d.g;
  PreWord W;
  const bool on = P.b > 0.0 && pre_word(d, g, P, W);
  const uint32_t base = pre_wave_word0(P);
  auto id_of = [&](int sl, int vt, int j, int& R, int& C) {
    pre_word_at(g, base + sl, R, C);
    C += j;
    return mid_id(g, R, C, vt);
  };
  auto free_one = [&](int sl, int vt, int j) {
    int R, C;
    return P.mid[id_of(sl, vt, j, R, C)] == 0;  // no lattice vertex sits on it
  };
  pre_deal(lds, on ? W.dh : 0u, on ? W.dv : 0u, pre_no_pay, [&](int sl, int vt, int j, uint32_t) {
    int R, C;
    const int64_t id = id_of(sl, vt, j, R, C);
    double mx, my;
    pre_mid_xy(g, R, C, vt, mx, my);
    pre_split_one<kAll>(P, g, id, mx, my);
  }, PreKeepIf<decltype(free_one)>{free_one});
}

// Slots of owner (k, i): Tb = [v, vdr, vdl] has sides E2 of v, E0 of vdl, E1 of
// v; Ta = [v, vr, vdr] has E0 of v, E1 of vr, E2 of v.  Bit j of a slot's
// sides: side j (corner j to corner j+1) is split.  fv / fr / fdl / fdr: the
// flags of v, vr, vdl and vdr (of the first three: the owners of the slot sides).
struct PreSlots {
  bool ok[2];
  uint32_t sides[2];
  bool moved[2];
  uint32_t fv, fr, fdl, fdr;
};
__device__ __forceinline__ uint32_t pre_slot_sides(int t, uint32_t fv, uint32_t fr, uint32_t fdl) {
  return t == 0 ? ((fv >> 2) & 1u) | ((fdl & 1u) << 1) | (((fv >> 1) & 1u) << 2)
                : (fv & 1u) | (((fr >> 1) & 1u) << 1) | (((fv >> 2) & 1u) << 2);
}
__device__ __forceinline__ PreSlots pre_owner_slots(const PreArgs& P, const Geo& g, int k, int i) {
  PreSlots S;
  const int o = k & 1;
  const int64_t v = (int64_t)k * g.NI + i, vd = (int64_t)(k + 1) * g.NI + i + o;  // vd: vdr
  S.ok[0] = pre_slot_ok(g, k, i, 0);
  S.ok[1] = pre_slot_ok(g, k, i, 1);
  S.fv = P.flags[v];
  S.fr = S.ok[1] ? P.flags[v + 1] : 0u;
  S.fdl = S.ok[0] ? P.flags[vd - 1] : 0u;
  S.fdr = (S.ok[0] || S.ok[1]) ? P.flags[vd] : 0u;
  const uint32_t fv = S.fv, fdr = S.fdr;
  S.sides[0] = S.ok[0] ? pre_slot_sides(0, fv, S.fr, S.fdl) : 0u;
  S.sides[1] = S.ok[1] ? pre_slot_sides(1, fv, S.fr, S.fdl) : 0u;
  S.moved[0] = S.ok[0] && ((fv | fdr | S.fdl) & kPreMoved);
  S.moved[1] = S.ok[1] && ((fv | S.fr | fdr) & kPreMoved);
  return S;
}
// One wave per row segment of kCB owners; lane l takes owners i0 + l + 64 j,
// j = 0 .. 3, so that loads and stores of neighbouring lanes are adjacent.
__device__ __forceinline__ bool pre_segment(const Geo& g, const Shared& sh, int64_t& seg, int& k, int& i0) {
  const uint32_t sg = blockIdx.x * 4u + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  seg = sg;
  if (seg >= sh.nseg) return false;
  const uint32_t kk = sg / (uint32_t)g.NCB;  // segment counts fit 32 bits (grid of nseg / 4 blocks)
  k = (int)kk;
  i0 = (int)(sg - kk * (uint32_t)g.NCB) * kCB;
  return true;
}

// Per row segment: inserted vertices (split sides owned) and triangles (one
// per slot, two for a slot with a split side).  The owners with a moved corner or a
// split side are gathered in LDS, their four corners' flags with them, and checked
// on full waves: the check's FP64 work was most of the kernel, done on waves with
// a few such owners each (with every place stored 8192 x 8192 344 -> 229 us, 4000 x
// 3000 72 -> 42; with computed ones 437 -> 242).
template <bool kAll>
__global__ void __launch_bounds__(256) k_pre_count(OneSrc src, PreArgs P, Shared sh) {
  __shared__ uint32_t lds[4][kCB];
  const Geo g = src.d.g;
  int64_t seg;
  int k, i0;
  if (!pre_segment(g, sh, seg, k, i0)) return;  // wave-uniform
  const int lane = threadIdx.x & 63;
  uint32_t* const item = lds[threadIdx.x >> 6];
  int ni = 0, nt = 0, n = 0;
  PreSlots S[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {  // every flag load of the lane first
    const int i = i0 + 64 * j + lane;
    S[j] = PreSlots{};
    if (i < g.NI) S[j] = pre_owner_slots(P, g, k, i);
  }
  const int o = k & 1;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    ni += __builtin_popcount(S[j].fv & 7u);
    bool look = false;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      nt += S[j].ok[t] ? (S[j].sides[t] ? 2 : 1) : 0;
      look |= S[j].moved[t] || S[j].sides[t];
    }
    const unsigned long long bal = __ballot(look);
    static_assert(kPreSnapped == 32, "six flag bits");
    if (look)
      item[n + lanes_below(bal)] = (uint32_t)(64 * j + lane) | ((S[j].fv & 63u) << 8) | ((S[j].fr & 63u) << 14) |
                                   ((S[j].fdl & 63u) << 20) | ((S[j].fdr & 63u) << 26);
    n += (int)__popcll(bal);
  }
  const int si = __builtin_amdgcn_readlane(wave_incl_scan_dpp(ni), 63);
  const int st = __builtin_amdgcn_readlane(wave_incl_scan_dpp(nt), 63);
  if (lane == 0) {
    sh.seg_cnt[seg] = make_int4(si, st, 0, 0);
    sh.seg_slow[seg] = 0ull;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  for (int q = lane; q < n; q += 64) {
    const uint32_t it = item[q];
    const int i = i0 + (int)(it & 255u);
    const uint32_t fv = (it >> 8) & 63u, fr = (it >> 14) & 63u, fdl = (it >> 20) & 63u, fdr = it >> 26;
    const bool ok[2] = {pre_slot_ok(g, k, i, 0), pre_slot_ok(g, k, i, 1)};
    // positive orientation of the base triangles after the moves, and of the two
    // triangles fanned around an inserted vertex; the four corners once for both
    const int64_t v = (int64_t)k * g.NI + i, vd = v + g.NI + o;
    const double2 A = pre_place<kAll>(P, g, v, k, i, fv), Br = pre_place<kAll>(P, g, ok[1] ? v + 1 : v, k, i + 1, fr),
                  Cl = pre_place<kAll>(P, g, ok[0] ? vd - 1 : v, k + 1, i + o - 1, fdl),
                  Dr = pre_place<kAll>(P, g, ok[0] || ok[1] ? vd : v, k + 1, i + o, fdr);
    auto area2 = [](double2 p, double2 q2, double2 r) {
      return (q2.x - p.x) * (r.y - p.y) - (q2.y - p.y) * (r.x - p.x);
    };
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      if (!ok[t]) continue;
      const uint32_t sides = pre_slot_sides(t, fv, fr, fdl);
      if (__builtin_popcount(sides) > 1) pre_error(P);  // a triangle with two split sides
      const double2 C1 = t == 0 ? Dr : Br, C2 = t == 0 ? Cl : Dr;
      if (!(area2(A, C1, C2) > 0.0)) pre_error(P);
      if (!sides) continue;
      const int js = __builtin_ctz(sides);
      const int64_t w = js == 1 ? (t == 0 ? vd - 1 : v + 1) : v;
      const int e = t == 0 ? (js == 0 ? 2 : (js == 1 ? 0 : 1)) : js;
      const int32_t m = P.split[3 * w + e];
      double2 M;
      pre_mid_xy(g, (m >> 1) / (g.CW + 2) - 1, (m >> 1) % (g.CW + 2) - 1, m & 1, M.x, M.y);
      const double2 a0 = pre_sel3(A, C1, C2, js), a1 = pre_sel3(C1, C2, A, js), a2 = pre_sel3(C2, A, C1, js);
      if (!(area2(a0, M, a2) > 0.0) || !(area2(M, a1, a2) > 0.0)) pre_error(P);
    }
  }
}

// Inserted vertices at their offsets (row segment base from the scan, owner
// offsets by wave scans), and the first inserted index of each owner that has one.
__global__ void __launch_bounds__(256) k_pre_inserted(OneSrc src, PreArgs P, Shared sh) {
  const Img& d = src.d;
  const Geo g = d.g;
  int64_t seg;
  int k, i0;
  if (!pre_segment(g, sh, seg, k, i0)) return;
  if (sh.seg_cnt[seg].x == 0) return;
  const int64_t nlat = (int64_t)g.NK * g.NI;
  int64_t base = sh.seg_off[seg].x;
  for (int j = 0; j < 4; ++j) {
    const int i = i0 + 64 * j + (int)(threadIdx.x & 63);
    const int64_t v = (int64_t)k * g.NI + i;
    const uint32_t f = i < g.NI ? (P.flags[v] & 7u) : 0u;
    const int n = __builtin_popcount(f);
    const int incl = wave_incl_scan_dpp(n);
    if (f) {
      int64_t pos = base + (incl - n);
      P.ins_base[v] = pos;
      for (int e = 0; e < 3; ++e) {
        if (!((f >> e) & 1u)) continue;
        const int32_t m = P.split[3 * v + e];
        const int R = (m >> 1) / (g.CW + 2) - 1, C = (m >> 1) % (g.CW + 2) - 1;
        double mx, my;
        pre_mid_xy(g, R, C, m & 1, mx, my);
        const int64_t id = nlat + pos++;
        if (id < P.vcap) {
          reinterpret_cast<double2*>(P.verts)[id] = make_double2(mx, my);
          if (P.on_polyline) P.on_polyline[id] = 1;
        }
      }
    }
    base += __builtin_amdgcn_readlane(incl, 63);
  }
}

// Triangles of each row segment at their offsets (row segment base from the
// scan, owner offsets by wave scans).  A slot with a split side j (corners a0 ->
// a1, opposite a2) becomes (a0, m, a2), (m, a1, a2) around the inserted vertex m
// (orientation checked by k_pre_count).  Per 64 owners the wave stages its
// triangles in LDS, as many ints from a 16-byte boundary there as they have in the
// output, and writes the full 16 bytes; what is left over begins the next round.
// 4000 x 3000: 104 -> 90 us, 3.7 TB/s.
__global__ void __launch_bounds__(256) k_pre_triangles(OneSrc src, PreArgs P, Shared sh) {
  __shared__ __attribute__((aligned(16))) int32_t stage[4][3 * 4 * 64 + 4];
  const Geo g = src.d.g;
  int64_t seg;
  int k, i0;
  if (!pre_segment(g, sh, seg, k, i0)) return;
  const int lane = (int)(threadIdx.x & 63);
  int32_t* const st = stage[threadIdx.x >> 6];
  const int32_t nlat = (int32_t)((int64_t)g.NK * g.NI);
  const int o = k & 1;
  const int64_t first = 3 * sh.seg_off[seg].y;  // the segment's first int
  // ints staged before this round's, from a 16-byte boundary of the output (those
  // before lo are another segment's)
  int a = (int)((((uintptr_t)P.tris >> 2) + (uintptr_t)first) & 3u), lo = a;
  int32_t* D = P.tris + (first - a);
  int64_t room = 3 * P.tcap - (first - a);  // ints from D that fit the capacity
  PreSlots SS[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {  // every flag load of the lane first
    const int i = i0 + 64 * j + lane;
    SS[j] = PreSlots{};
    if (i < g.NI) SS[j] = pre_owner_slots(P, g, k, i);
  }
  // the inserted vertices of the split sides, all in flight at once: asked for
  // where they are used they were eight waits one after the other
  const int32_t* const ins = reinterpret_cast<const int32_t*>(P.ins_base);  // low words
  int32_t mid[4][2];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      // the owner of side js
      const int js = __builtin_ctz(SS[j].sides[t] | 8u);
      const int64_t v = (int64_t)k * g.NI + i0 + 64 * j + lane;
      const int64_t w = js == 1 ? (t == 0 ? v + g.NI + o - 1 : v + 1) : v;
      mid[j][t] = ins[SS[j].sides[t] ? 2 * w : 0];
    }
  }
  auto wave_sync = [] {  // the wave's LDS writes are seen by its own later reads
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int i = i0 + 64 * j + lane;
    const PreSlots& S = SS[j];
    int nt = 0;
#pragma unroll
    for (int t = 0; t < 2; ++t) nt += S.ok[t] ? (S.sides[t] ? 2 : 1) : 0;
    const int incl = wave_incl_scan_dpp(nt);
    const int total = a + 3 * __builtin_amdgcn_readlane(incl, 63);
    if (nt) {
      Tri3* at = reinterpret_cast<Tri3*>(st + a + 3 * (incl - nt));
      auto put = [&](int32_t x, int32_t y, int32_t z) {
        Tri3 t3;
        t3.a = x;
        t3.b = y;
        t3.c = z;
        *at++ = t3;
      };
      const int32_t v = (int32_t)((int64_t)k * g.NI + i), vd = v + g.NI + o;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        if (!S.ok[t]) continue;
        const int32_t C1 = t == 0 ? vd : v + 1, C2 = t == 0 ? vd - 1 : vd;
        if (!S.sides[t]) {
          put(v, C1, C2);
          continue;
        }
        const int js = __builtin_ctz(S.sides[t]);
        // its owned side at its owner
        const int e = t == 0 ? (js == 0 ? 2 : (js == 1 ? 0 : 1)) : js;
        const uint32_t fw = js == 1 ? (t == 0 ? S.fdl : S.fr) : S.fv;
        const int32_t m = nlat + mid[j][t] + __builtin_popcount(fw & ((1u << e) - 1u));
        const int32_t a0 = pre_sel3(v, C1, C2, js), a1 = pre_sel3(C1, C2, v, js), a2 = pre_sel3(C2, v, C1, js);
        put(a0, m, a2);
        put(m, a1, a2);
      }
    }
    wave_sync();
    const int full = total >> 2;
    for (int q = lane; q < full; q += 64) {
      const int4 x = *reinterpret_cast<const int4*>(st + 4 * q);
      if (4 * q >= lo && 4 * q + 4 <= room) {
        *reinterpret_cast<int4*>(D + 4 * q) = x;
      } else {
        const int32_t xs[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (4 * q + c >= lo && 4 * q + c < room) D[4 * q + c] = xs[c];
      }
    }
    const int32_t left = lane < 4 ? st[4 * full + lane] : 0;
    wave_sync();
    if (lane < 4) st[lane] = left;
    D += 4 * full;
    room -= 4 * full;
    a = total & 3;
    if (full) lo = 0;
  }
  if (lane >= lo && lane < a && lane < room) D[lane] = st[lane];
}

__global__ void k_pre_clear(PreArgs P, int64_t nmid, int64_t nown) {
  uint32_t* m4 = reinterpret_cast<uint32_t*>(P.mid);  // the region is padded to 256 bytes
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < (nmid + 3) / 4; q += (int64_t)gridDim.x * blockDim.x)
    m4[q] = 0u;
  for (int q = threadIdx.x; blockIdx.x == 0 && q < kPreCounts; q += blockDim.x) P.counts[q] = 0;
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < P.ntouched; q += (int64_t)gridDim.x * blockDim.x)
    P.touched[q] = 0u;
  uint32_t* f4 = reinterpret_cast<uint32_t*>(P.flags);  // padded to 256 bytes
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < (nown + 3) / 4; q += (int64_t)gridDim.x * blockDim.x)
    f4[q] = 0u;
  if (P.used) {
    uint32_t* u4 = reinterpret_cast<uint32_t*>(P.used);  // padded to 256 bytes
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < (P.usedcap + 3) / 4;
         q += (int64_t)gridDim.x * blockDim.x)
      u4[q] = 0u;
  }
}

__global__ void k_pre_sizes(OneSrc src, PreArgs P, Shared sh, int64_t* out) {
  const Geo g = src.d.g;
  const longlong4 tot = sh.seg_off[sh.nseg];
  int64_t ns = 0, nr = 0;  // one wave
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    ns += P.counts[kPreTally + 64 * q + threadIdx.x];
    nr += P.counts[kPreTally + 256 + 64 * q + threadIdx.x];
  }
  for (int off = 32; off > 0; off >>= 1) {
    ns += __shfl_xor(ns, off);
    nr += __shfl_xor(nr, off);
  }
  if (threadIdx.x) return;
  out[0] = (int64_t)g.NK * g.NI + tot.x;  // vertices
  out[1] = tot.y;                          // triangles
  out[2] = ns;                             // snapped
  out[3] = nr;                             // repelled
  out[4] = tot.x;                          // inserted
  out[5] = P.counts[2] ? SBMT_E_PROTOCOL : ((out[0] > P.vcap || out[1] > P.tcap) ? SBMT_E_CAPACITY : SBMT_OK);
  if (out[0] > 0x7fffffffLL) out[5] = SBMT_E_INDEX_OVERFLOW;
}

// ---------------------------------------------------------------------------
// Retriangulation of the preprocessed grid against the polyline (the mesh of
// Alg. 3, Sec. 3.5): every grid triangle is cut by the polyline pieces inside
// it, its faces are traced along its boundary and the pieces, and the
// foreground faces are triangulated by the template rule (fanned from the
// chain vertex inside the triangle; the quadrilateral between two chords split
// by the diagonal joining their exits; else fanned from the face's earliest
// chain point); an uncut triangle is kept whole when it lies in the foreground.
// Decisions in FP64 on the moved points, as the oracle takes them; the margins
// c and b of Steps 2 and 3 keep them away from zero.  A corner that sits on a
// polyline vertex is that vertex by identity.
//
// Output vertices: the grid vertices (ids 0 .. NV-1, positions from the grid
// phase), then per owner (by the scan) its new vertices: the crossings of the
// grid edges it owns, edge slot by edge slot (slot 2e and 2e+1: side E_e, or
// its two halves around the inserted vertex; slot 6 + t: the fan edge of its
// split slot t), each edge's crossings in order from its lower-numbered end;
// then the polyline vertices strictly inside its slots' triangles.
// ---------------------------------------------------------------------------
struct PreSeg {
  double px, py, qx, qy;
  int32_t jp, jq;  // ids of the polyline vertices at the start and the end
};
__device__ __forceinline__ int32_t pre_cell_edge_mid(const Geo& g, int R, int C, int e) {
  // cell edges: 0 top, 1 right, 2 bottom, 3 left
  return (int32_t)(e == 0 ? mid_id(g, R, C, 0) : (e == 1 ? mid_id(g, R, C + 1, 1) : (e == 2 ? mid_id(g, R + 1, C, 0) : mid_id(g, R, C, 1))));
}
// A thread's copy of the coarse samples around one owner: rows R0 .. R0+nr-1,
// columns C0 .. C0+31 as row masks (background outside the stored raster).
struct PreBits {
  int R0, C0, nr;
  uint32_t rw[6];
};
__device__ __forceinline__ void pre_bits_load(const Img& d, const Geo& g, int R0, int C0, int nr, PreBits& B) {
  B.R0 = R0;
  B.C0 = C0;
  B.nr = nr;
  const int cc = C0 + kRingC;
  const int w0 = cc >> 5, sh = cc & 31;
#pragma unroll
  for (int r = 0; r < 6; ++r) {
    const int R = R0 + r;
    uint32_t w = 0;
    if (r < nr && R >= 0 && R < g.CH) {
      const uint32_t* row = d.bits + (int64_t)(R + kRing) * g.wpr;
      const uint64_t lo = (w0 >= 0 && w0 < g.wpr) ? row[w0] : 0u;
      const uint64_t hi = (w0 + 1 >= 0 && w0 + 1 < g.wpr) ? row[w0 + 1] : 0u;
      w = (uint32_t)((((hi << 32) | lo) >> sh));
      // columns outside the image are background
      const int cfirst = C0, clast = C0 + 31;
      if (cfirst < 0) w = -cfirst >= 32 ? 0u : (w & (~0u << (-cfirst)));
      if (clast >= g.CW) w &= (g.CW - C0) <= 0 ? 0u : (g.CW - C0 >= 32 ? ~0u : ((1u << (g.CW - C0)) - 1u));
    }
    B.rw[r] = w;
  }
}
// Row r of the block, selected rather than indexed (which would put rw in
// scratch memory).
__device__ __forceinline__ uint32_t pre_bits_row(const PreBits& B, int r) {
  uint32_t w = B.rw[0];
#pragma unroll
  for (int q = 1; q < 6; ++q) w = r == q ? B.rw[q] : w;
  return w;
}
__device__ __forceinline__ int pre_cell_case(const Img& d, const Geo& g, int R, int C, const PreBits* B = nullptr) {
  if (B && R >= B->R0 && R + 1 < B->R0 + B->nr && C >= B->C0 && C + 1 < B->C0 + 32) {
    const uint32_t t = pre_bits_row(*B, R - B->R0) >> (C - B->C0), u = pre_bits_row(*B, R + 1 - B->R0) >> (C - B->C0);
    return (int)((t & 1u) | ((t & 2u)) | ((u & 2u) << 1) | ((u & 1u) << 3));
  }
  return sample_at(d, g, R, C) | (sample_at(d, g, R, C + 1) << 1) | (sample_at(d, g, R + 1, C + 1) << 2) |
         (sample_at(d, g, R + 1, C) << 3);
}
// Calls f(seg) for every segment of the dual cells that contain a point of
// [x0, x1] x [y0, y1] (callers widen their boxes by a margin, so a cell that
// only touches the box's border holds no segment reaching inside it).  A lane
// skips its empty cells in an inner loop of integer work and all lanes meet at
// f, whose FP64 work then runs once per segment of the lane with the most (a
// walk in step over the cells would run it for every cell and segment slot
// that is present in any lane).
template <class F>
__device__ __forceinline__ void pre_segs_in_box(const Img& d, const Geo& g, double x0, double x1, double y0, double y1, F f,
                                                const PreBits* B = nullptr) {
  const int R0 = floor_index(g, y0), R1 = floor_index(g, y1);
  const int C0 = floor_index(g, x0), C1 = floor_index(g, x1);
  int R = R0, C = C0, Rc = R0, Cc = C0, j = 0;  // the cell to look at next; the cell at hand and its next segment
  uint32_t ms = 0;
  for (;;) {
    while (j >= (int)(ms & 3u) && R <= R1) {
      const int cs = C <= C1 ? pre_cell_case(d, g, R, C, B) : 0;
      ms = cs == 0 || cs == 15 ? 0u : ms_case(cs);
      j = 0;
      Rc = R;
      Cc = C;
      const bool end = C >= C1;
      C = end ? C0 : C + 1;
      R = end ? R + 1 : R;
    }
    if (j >= (int)(ms & 3u)) break;
    PreSeg S;
    cell_segment(g, Rc, Cc, ms, j, S.px, S.py, S.qx, S.qy);
    S.jp = pre_cell_edge_mid(g, Rc, Cc, (int)((ms >> (2 + 4 * j)) & 3u));
    S.jq = pre_cell_edge_mid(g, Rc, Cc, (int)((ms >> (4 + 4 * j)) & 3u));
    f(S);
    ++j;
  }
}
// Inside the foreground: the dual cell of the point, uniform or left of each
// of its segments (segments have the foreground on their left).  Used for
// points at a distance from the polyline (lattice corners off it, centroids of
// uncut triangles).
__device__ __forceinline__ int pre_inside_point(const Img& d, const Geo& g, double x, double y,
                                                const PreBits* B = nullptr) {
  const int R = floor_index(g, y), C = floor_index(g, x);
  const int cs = pre_cell_case(d, g, R, C, B);
  if (cs == 0 || cs == 15) return cs == 15;
  const uint32_t ms = ms_case(cs);
  for (int j = 0; j < (int)(ms & 3u); ++j) {
    double px, py, qx, qy;
    cell_segment(g, R, C, ms, j, px, py, qx, qy);
    if (!((qx - px) * (y - py) - (qy - py) * (x - px) > 0.0)) return 0;
  }
  return 1;
}
// Grid vertex: id, position, the polyline vertex it sits on (or -1).  Grid
// vertex and owner indices fit 32 bits (the entry points check it).
struct PreGV {
  int32_t id;
  int32_t bnd;
  double x, y;
};
__device__ __forceinline__ PreGV pre_lat_gv(const PreArgs& P, const Geo& g, int k, int i) {
  PreGV r;
  const int64_t v = (int64_t)k * g.NI + i;
  r.id = (int32_t)v;
  const uint32_t f = P.flags[v];
  const double2 p = pre_place<false>(P, g, v, k, i, f);
  r.x = p.x;
  r.y = p.y;
  r.bnd = (f & kPreSnapped) ? P.snap_mid[v] : -1;
  return r;
}
// The vertex inserted on side e of owner w (flags fw).
__device__ __forceinline__ PreGV pre_ins_gv(const PreArgs& P, const Geo& g, int64_t w, int e, uint32_t fw) {
  PreGV r;
  r.id = (int32_t)((int64_t)g.NK * g.NI + P.ins_base[w] + __builtin_popcount(fw & ((1u << e) - 1u)));
  const double2 p = reinterpret_cast<const double2*>(P.verts)[r.id];
  r.x = p.x;
  r.y = p.y;
  r.bnd = P.split[3 * w + e];
  return r;
}
// Whether segment S crosses the grid edge U - W at an interior point of both
// (a segment end that is U's or W's polyline vertex lies on the edge's line);
// te: the crossing's position along U -> W (monotone, unnormalised).
__device__ __forceinline__ bool pre_crosses(const PreSeg& S, const PreGV& U, const PreGV& W, double* te) {
  const double gx = W.x - U.x, gy = W.y - U.y;
  const double dp = (S.jp == U.bnd || S.jp == W.bnd) ? 0.0 : gx * (S.py - U.y) - gy * (S.px - U.x);
  const double dq = (S.jq == U.bnd || S.jq == W.bnd) ? 0.0 : gx * (S.qy - U.y) - gy * (S.qx - U.x);
  if (!((dp > 0.0 && dq < 0.0) || (dp < 0.0 && dq > 0.0))) return false;
  const double hx = S.qx - S.px, hy = S.qy - S.py;
  const double eu = hx * (U.y - S.py) - hy * (U.x - S.px), ew = hx * (W.y - S.py) - hy * (W.x - S.px);
  if (!((eu > 0.0 && ew < 0.0) || (eu < 0.0 && ew > 0.0))) return false;
  if (te) {
    const double t = dp / (dp - dq);
    *te = (S.px + t * hx - U.x) * gx + (S.py + t * hy - U.y) * gy;
  }
  return true;
}
// The crossing point of grid edge (lo, hi), lo < hi, by segment S.
__device__ __forceinline__ void pre_crossing_xy(const PreSeg& S, const PreGV& L, const PreGV& H, double& x, double& y) {
  const double gx = H.x - L.x, gy = H.y - L.y;
  const double dp = gx * (S.py - L.y) - gy * (S.px - L.x);
  const double dq = gx * (S.qy - L.y) - gy * (S.qx - L.x);
  const double t = dp / (dp - dq);
  x = S.px + t * (S.qx - S.px);
  y = S.py + t * (S.qy - S.py);
}
// Calls f(seg, te) for every segment crossing grid edge U - W.
template <class F>
__device__ __forceinline__ void pre_edge_crossings(const Img& d, const Geo& g, const PreGV& U, const PreGV& W, F f,
                                                   const PreBits* B = nullptr) {
  const double m = 1e-9;
  pre_segs_in_box(d, g, fmin(U.x, W.x) - m, fmax(U.x, W.x) + m, fmin(U.y, W.y) - m, fmax(U.y, W.y) + m,
                  [&](const PreSeg& S) {
                    double te;
                    if (pre_crosses(S, U, W, &te)) f(S, te);
                  }, B);
}

// A grid triangle of an owner's slot: corners, and per edge e (corner e to
// e+1) the owner and edge slot that number its crossings.
struct PreGT {
  PreGV c[3];
  int32_t eo[3];
  int es[3];
};
// Edge slot q of owner (k, i): its ends (false if the owner has no such edge).
__device__ bool pre_edge_slot(const PreArgs& P, const Geo& g, int k, int i, const PreSlots& S, int q, PreGV& A,
                              PreGV& B) {
  const int o = k & 1;
  const int64_t v = (int64_t)k * g.NI + i;
  if (q < 6) {
    const int e = q >> 1;
    if (!pre_edge_live(g, k, i, e)) return false;
    const int kw = e == 0 ? k : k + 1, iw = e == 0 ? i + 1 : (e == 1 ? i + o - 1 : i + o);
    const bool split = (S.fv >> e) & 1u;
    if (!split && (q & 1)) return false;
    const PreGV U = pre_lat_gv(P, g, k, i), W = pre_lat_gv(P, g, kw, iw);
    if (!split) {
      A = U;
      B = W;
      return true;
    }
    const PreGV M = pre_ins_gv(P, g, v, e, S.fv);
    A = (q & 1) ? M : U;
    B = (q & 1) ? W : M;
    return true;
  }
  const int t = q - 6;
  if (!S.ok[t] || !S.sides[t]) return false;
  const int js = __builtin_ctz(S.sides[t]);
  const int64_t C2 = t == 0 ? (int64_t)(k + 1) * g.NI + (i + o - 1) : (int64_t)(k + 1) * g.NI + (i + o);
  const int64_t w = t == 0 ? (js == 1 ? C2 : v) : (js == 1 ? v + 1 : v);
  const int e = t == 0 ? (js == 0 ? 2 : (js == 1 ? 0 : 1)) : js;
  const uint32_t fw = t == 0 ? (js == 1 ? S.fdl : S.fv) : (js == 1 ? S.fr : S.fv);
  A = pre_ins_gv(P, g, w, e, fw);
  const int jc = (js + 2) % 3;  // the corner opposite the split side
  B = pre_lat_gv(P, g, jc == 0 || (jc == 1 && t == 1) ? k : k + 1,
                 jc == 0 ? i : (t == 0 ? i + o - (jc - 1) : (jc == 1 ? i + 1 : i + o)));
  return true;
}
// The grid triangles of slot t of owner (k, i): one, or two fanned around the
// inserted vertex of its split side.  Returns their number.
__device__ int pre_slot_tris(const PreArgs& P, const Geo& g, int k, int i, const PreSlots& S, int t, PreGT* T) {
  if (!S.ok[t]) return 0;
  const int o = k & 1;
  const int64_t v = (int64_t)k * g.NI + i;
  const int64_t C2 = t == 0 ? (int64_t)(k + 1) * g.NI + (i + o - 1) : (int64_t)(k + 1) * g.NI + (i + o);
  // side j: owner, owned side, and whether corner j is that owner
  // Tb = [v, vdr, vdl]: E2 of v, E0 of vdl, E1 of v; Ta = [v, vr, vdr]: E0 of v, E1 of vr, E2 of v
  const int64_t so0 = v, so1 = t == 0 ? C2 : v + 1, so2 = v;
  const int se0 = t == 0 ? 2 : 0, se1 = t == 0 ? 0 : 1, se2 = t == 0 ? 1 : 2;
  const bool sa0 = true, sa1 = t != 0, sa2 = false;
  const PreGV G0 = pre_lat_gv(P, g, k, i), G1 = pre_lat_gv(P, g, t == 0 ? k + 1 : k, t == 0 ? i + o : i + 1),
              G2 = pre_lat_gv(P, g, k + 1, t == 0 ? i + o - 1 : i + o);
  if (!S.sides[t]) {
    T[0].c[0] = G0;
    T[0].c[1] = G1;
    T[0].c[2] = G2;
    T[0].eo[0] = so0;
    T[0].eo[1] = so1;
    T[0].eo[2] = so2;
    T[0].es[0] = 2 * se0;
    T[0].es[1] = 2 * se1;
    T[0].es[2] = 2 * se2;
    return 1;
  }
  const int js = __builtin_ctz(S.sides[t]);
  const uint32_t fw = t == 0 ? (js == 1 ? S.fdl : S.fv) : (js == 1 ? S.fr : S.fv);
  const int j1 = (js + 1) % 3, j2 = (js + 2) % 3;
  const int64_t soj = pre_sel3(so0, so1, so2, js);
  const int sej = pre_sel3(se0, se1, se2, js);
  const bool saj = pre_sel3(sa0, sa1, sa2, js);
  const PreGV M = pre_ins_gv(P, g, soj, sej, fw);
  const int h0 = 2 * sej + (saj ? 0 : 1), h1 = 2 * sej + (saj ? 1 : 0);
  const PreGV Gs = pre_sel3(G0, G1, G2, js), G1s = pre_sel3(G0, G1, G2, j1), G2s = pre_sel3(G0, G1, G2, j2);
  // (a0, m, a2): a0 -> m (half of the split side), m -> a2 (fan edge), a2 -> a0
  T[0].c[0] = Gs;
  T[0].c[1] = M;
  T[0].c[2] = G2s;
  T[0].eo[0] = soj;
  T[0].es[0] = h0;
  T[0].eo[1] = v;
  T[0].es[1] = 6 + t;
  T[0].eo[2] = pre_sel3(so0, so1, so2, j2);
  T[0].es[2] = 2 * pre_sel3(se0, se1, se2, j2);
  // (m, a1, a2): m -> a1 (other half), a1 -> a2, a2 -> m (fan edge)
  T[1].c[0] = M;
  T[1].c[1] = G1s;
  T[1].c[2] = G2s;
  T[1].eo[0] = soj;
  T[1].es[0] = h1;
  T[1].eo[1] = pre_sel3(so0, so1, so2, j1);
  T[1].es[1] = 2 * pre_sel3(se0, se1, se2, j1);
  T[1].eo[2] = v;
  T[1].es[2] = 6 + t;
  return 2;
}

// Per-owner counts of the retriangulation: crossings of edge slot q in bits
// 2q .. 2q+1, polyline vertices inside its triangles in 16 .. 18, output
// triangles in 19 .. 26, cut grid triangles in 27 .. 29.
__device__ __forceinline__ int pre_rc_cross(uint32_t rc, int q) { return (int)((rc >> (2 * q)) & 3u); }
__device__ __forceinline__ int pre_rc_before(uint32_t rc, int q) {  // crossings of slots before q
  int n = 0;
  for (int j = 0; j < q; ++j) n += pre_rc_cross(rc, j);
  return n;
}
__device__ __forceinline__ int pre_rc_inner(uint32_t rc) { return (int)((rc >> 16) & 7u); }
__device__ __forceinline__ int pre_rc_tris(uint32_t rc) { return (int)((rc >> 19) & 255u); }
__device__ __forceinline__ int pre_rc_cut(uint32_t rc) { return (int)((rc >> 27) & 7u); }
constexpr uint32_t kPrePlain = 1u << 31;  // a touched owner of two slots without a split side
// A grid vertex's id in the mesh (of one that is used).
__device__ __forceinline__ int32_t pre_vertex(const PreArgs& P, int64_t v) {
  const PreUsed u = P.uword[v >> 6];
  return (int32_t)P.vbsum[v / kPreVScan] + u.base + (int32_t)__popcll(u.bits & ((1ull << (v & 63)) - 1ull));
}
// The counts of an owner, zero of one that no segment can reach.
__device__ __forceinline__ uint32_t pre_owner_counts(const PreArgs& P, const Geo& g, uint32_t w) {
  const uint32_t k = w / (uint32_t)g.NI, i = w - k * (uint32_t)g.NI;
  return (P.touched[(int64_t)k * 8 * g.NCB + (i >> 5)] >> (i & 31u)) & 1u ? P.rcount[w] : 0u;
}

struct PreSub {
  PreSeg S;
  double t0, t1;
  int e0, e1, c0, c1;
};

// Owners whose slot triangles a segment can reach: every segment marks the
// owners whose slot box on the lattice, widened by a + b (the moves and the
// inserted vertices stay within it), meets the segment's box.  An unmarked
// owner is quiet: its triangles are uncut, its corners are lattice vertices
// off the polyline, and the inside label of the owner vertex decides them.
// One bit per owner: a row of a segment's box is one or two words, set without
// a look at what is there (a byte each, loaded and set by an atomic, took
// 520 us on 0.9 M segments; now 100 us).
__device__ void pre_touch_seg(const PreArgs& P, const Geo& g, double px, double py, double qx, double qy) {
  const double r = widen(P.a + P.b) + 1e-9, hx = pre_hx(g);
  const double x0 = fmin(px, qx) - r, x1 = fmax(px, qx) + r, y0 = fmin(py, qy) - r, y1 = fmax(py, qy) + r;
  for (int k = max(0, pre_row_floor(g, y0) - 1); k <= min(g.NK - 1, pre_row_floor(g, y1)); ++k) {
    const int ia = max(0, (int)__builtin_floor(pre_col(g, k, x0 - hx)));
    const int ib = min(g.NI - 1, (int)__builtin_floor(pre_col(g, k, x1 + 0.5 * hx)) + 1);
    if (ia > ib) continue;
    uint32_t* const row = P.touched + (int64_t)k * 8 * g.NCB;
    for (int w = ia >> 5; w <= ib >> 5; ++w) {
      const uint32_t lo = w == ia >> 5 ? ~0u << (ia & 31) : ~0u, hi = w == ib >> 5 ? ~0u >> (31 - (ib & 31)) : ~0u;
      atomicOr(row + w, lo & hi);
    }
  }
}
// The touched bits of the 64 owners of step j of a row segment.
__device__ __forceinline__ unsigned long long pre_touched64(const PreArgs& P, int64_t seg, int j) {
  const uint2 w = reinterpret_cast<const uint2*>(P.touched)[4 * seg + j];
  return (unsigned long long)w.x | ((unsigned long long)w.y << 32);
}
__global__ void __launch_bounds__(256) k_pre_mesh_touch(OneSrc src, PreArgs P) {
  __shared__ uint16_t lds[4][kPreDeal];
  const Img& d = src.d;
  const Geo g = d.g;
  PreWord W;
  const bool on = pre_word(d, g, P, W);
  const uint32_t cells = on ? (W.dh | W.dv | (W.cur ^ W.b1)) : 0u;
  const uint32_t base = pre_wave_word0(P);
  auto cs_of = [&](int, int j) {
    return ((W.cur >> j) & 1u) | (((W.c1 >> j) & 1u) << 1) | (((W.b1 >> j) & 1u) << 2) | (((W.bel >> j) & 1u) << 3);
  };
  pre_deal(lds, cells, 0u, cs_of, [&](int sl, int, int j, uint32_t cs) {
    int R, C0;
    pre_word_at(g, base + sl, R, C0);
    const uint32_t ms = ms_case((int)cs);
    for (int q = 0; q < (int)(ms & 3u); ++q) {
      double px, py, qx, qy;
      cell_segment(g, R, C0 + j, ms, q, px, py, qx, qy);
      pre_touch_seg(P, g, px, py, qx, qy);
    }
  });
}

// The samples around owner (k, i): the box of its two slots on the lattice
// widened by a + b (every moved or inserted corner stays in it), with the
// cells the enumerations of its edges and triangles look at (one more row and
// column on each side).
__device__ __forceinline__ void pre_owner_bits(const Img& d, const Geo& g, const PreArgs& P, int k, int i, PreBits& B) {
  const double hx = pre_hx(g), lx = lat_x(g, pre_lat_X(g, k, i));
  const double r = widen(P.a + P.b) + 1e-9;
  const int R0 = floor_index(g, lat_y(g, k) - r) - 1, R1 = floor_index(g, lat_y(g, k + 1) + r) + 1;
  const int C0 = floor_index(g, lx - 0.5 * hx - r) - 1;
  pre_bits_load(d, g, R0, C0, min(6, R1 - R0 + 1), B);
}

// Grid triangle z (slot z / 2, its z % 2-th triangle) of owner (k, i).
__device__ __forceinline__ bool pre_owner_tri(const PreArgs& P, const Geo& g, int k, int i, const PreSlots& S, int z,
                                              PreGT& T) {
  PreGT TT[2];
  const int m = pre_slot_tris(P, g, k, i, S, z >> 1, TT);
  if ((z & 1) >= m) return false;
  if (z & 1)  // constant indices keep TT in registers
    T = TT[1];
  else
    T = TT[0];
  return true;
}

// The slot of cut grid triangle z of list position t in the kept outputs.
__device__ __forceinline__ int64_t pre_cut_slot(const PreArgs& P, int64_t t, int z, uint32_t rt) {
  return (int64_t)P.cbase[t] + __builtin_popcount((rt >> 28) & ((1u << z) - 1u));
}

// The touched owners of each row segment (their list offsets come from a
// scan), a thread each.
__global__ void __launch_bounds__(256) k_pre_mesh_tcount(PreArgs P, Shared sh) {
  const int64_t seg = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (seg >= sh.nseg) return;
  int n = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) n += (int)__popcll(pre_touched64(P, seg, j));
  sh.seg_cnt[seg] = make_int4(n, 0, 0, 0);
  sh.seg_slow[seg] = 0ull;
}

// Quiet owners: their slots are kept whole when the owner vertex is inside, a bit
// each; the touched ones go to the list at their segment's offset, their counts
// cleared for the dense pass.
__global__ void __launch_bounds__(256) k_pre_mesh_count(OneSrc src, PreArgs P, Shared sh) {
  const Img& d = src.d;
  const Geo g = d.g;
  int64_t seg;
  int k, i0;
  if (!pre_segment(g, sh, seg, k, i0)) return;  // wave-uniform
  const int lane = threadIdx.x & 63;
  const double y = lat_y(g, k);
  int64_t at = sh.seg_off[seg].x;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int i = i0 + 64 * j + lane;
    const int64_t v = (int64_t)k * g.NI + i;
    const unsigned long long bal = pre_touched64(P, seg, j);  // uniform
    const bool touched = (bal >> lane) & 1ull;
    if (touched) {
      P.tlist[at + lanes_below(bal)] = (int32_t)v;
      P.rcount[v] = 0u;
      P.rtri[v] = 0u;
    }
    const bool tb = i < g.NI && pre_slot_ok(g, k, i, 0), ta = i < g.NI && pre_slot_ok(g, k, i, 1);
    const bool in = !touched && (tb || ta) && pre_inside_point(d, g, lat_x(g, pre_lat_X(g, k, i)), y);
    if (in) {  // the corners of its slots are in the mesh
      const int64_t vd = v + g.NI + (k & 1);
      P.used[v] = 1;
      P.used[vd] = 1;
      if (tb) P.used[vd - 1] = 1;
      if (ta) P.used[v + 1] = 1;
    }
    const unsigned long long ins = __ballot(in);
    if (lane == 0) P.inside[4 * seg + j] = ins;
    at += (int64_t)__popcll(bal);
  }
}

// Work over n items in chunks of a block (a grid-stride loop): light(item)
// runs each item and returns true to put it off; put-off items are gathered
// in LDS and run by heavy(item) on full blocks, the rest at the end.  dl
// holds 2 * 256 entries; *nd starts at 0.
template <class Light, class Heavy>
__device__ __forceinline__ void pre_dense(int64_t n, int64_t* dl, int* nd, Light light, Heavy heavy) {
  for (int64_t base = (int64_t)blockIdx.x * 256;; base += (int64_t)gridDim.x * 256) {
    const bool more = base < n;  // uniform
    if (more) {
      const int64_t it = base + threadIdx.x;
      if (it < n && light(it)) dl[atomicAdd(nd, 1)] = it;
    }
    __syncthreads();
    int m = *nd;
    while (m >= 256 || (!more && m > 0)) {  // uniform
      const int take = m >= 256 ? 256 : m;
      if ((int)threadIdx.x < take) heavy(dl[m - take + threadIdx.x]);
      m -= take;
      __syncthreads();
    }
    if (threadIdx.x == 0) *nd = m;
    __syncthreads();
    if (!more) break;
  }
}
__device__ __forceinline__ void pre_tl_owner(const Geo& g, const PreArgs& P, int64_t t, int& k, int& i) {
  const uint32_t v = (uint32_t)P.tlist[t];
  const uint32_t kk = v / (uint32_t)g.NI;
  k = (int)kk;
  i = (int)(v - kk * (uint32_t)g.NI);
}

// Counts of a cut grid triangle of a touched owner: its triangles, inner vertex
// and the cut are added to the owner's words.
__device__ __forceinline__ void pre_add_counts(const PreArgs& P, int64_t v, int z, int nt, int nin) {
  atomicOr(&P.rtri[v], ((uint32_t)nt << (6 * z)) | ((uint32_t)nin << (24 + z)));
  atomicAdd(&P.rcount[v], ((uint32_t)nin << 16) | ((uint32_t)nt << 19) | (1u << 27));
}
// Counts of the touched owners.  The plain ones (both base triangles there and
// no split side: nine in ten) take k_pre_mesh_probe_plain, one lane per owner:
// its four corners and its raster words are loaded once, together, and every
// segment around it is looked at once, for its two triangles (the segment
// clipped against each: an uncut triangle counts as one when in the foreground,
// a cut one gets its cut bit and is counted by k_pre_mesh_cut_count) and its
// three edges (crossings); its words are written without atomics.  The others
// are marked kPreTodo and gathered by k_pre_mesh_probe_owner, which takes their
// four grid triangles and eight edge slots one by one, with the loads of each.
// Taking every owner that way was bound by the latency of those loads, about
// thirty in a row (2.26 ms on 77 M owners; now 0.78 + 0.52 ms).
constexpr uint32_t kPreTodo = 1u << 24;  // (an inner vertex without a cut triangle: no count leaves that)

// Sides of a segment's ends on the line through A -> B (a segment end that is
// the polyline vertex of A or B lies on it).
__device__ __forceinline__ void pre_half(const PreSeg& S, double2 A, double2 B, int32_t ba, int32_t bb, double& fp,
                                         double& fq) {
  fp = (ba == S.jp || bb == S.jp) ? 0.0 : (B.x - A.x) * (S.py - A.y) - (B.y - A.y) * (S.px - A.x);
  fq = (ba == S.jq || bb == S.jq) ? 0.0 : (B.x - A.x) * (S.qy - A.y) - (B.y - A.y) * (S.qx - A.x);
}
// The part of segment S inside the triangle of corners c, whose edges' sides of
// S's ends are fp, fq: 1 if it cuts the triangle (its parameters, and the edge
// or corner at each end, to *sub if given), 0 if not; a segment that joins two
// corners cuts nothing and sets side (the triangle left of it: 1, right: 0).
__device__ __forceinline__ int pre_clip(const PreSeg& S, const double2 (&c)[3], const int32_t (&bnd)[3],
                                        const double (&fp)[3], const double (&fq)[3], int& side, PreSub* sub = nullptr) {
  const double m = 1e-9;
  if (fmax(S.px, S.qx) < fmin(c[0].x, fmin(c[1].x, c[2].x)) - m || fmin(S.px, S.qx) > fmax(c[0].x, fmax(c[1].x, c[2].x)) + m ||
      fmax(S.py, S.qy) < fmin(c[0].y, fmin(c[1].y, c[2].y)) - m || fmin(S.py, S.qy) > fmax(c[0].y, fmax(c[1].y, c[2].y)) + m)
    return 0;
  double t0 = 0.0, t1 = 1.0;
  int e0 = -1, e1 = -1;
  bool out = false;
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    out = out || (fp[e] < 0 && fq[e] < 0);
    if (!(fp[e] < 0 && fq[e] < 0) && !(fp[e] >= 0 && fq[e] >= 0)) {
      const double t = fp[e] / (fp[e] - fq[e]);
      if (fp[e] < 0) {
        e0 = t > t0 ? e : e0;
        t0 = t > t0 ? t : t0;
      } else {
        e1 = t < t1 ? e : e1;
        t1 = t < t1 ? t : t1;
      }
    }
  }
  if (out || !(t1 > t0)) return 0;
  int c0 = -1, c1 = -1;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    if (bnd[j] == S.jp && t0 == 0.0) c0 = j;
    if (bnd[j] == S.jq && t1 == 1.0) c1 = j;
  }
  if (c0 >= 0 && c1 >= 0) {
    const double2 T3 = pre_sel3(c[0], c[1], c[2], 3 - c0 - c1);
    side = ((S.qx - S.px) * (T3.y - S.py) - (S.qy - S.py) * (T3.x - S.px)) > 0 ? 1 : 0;
    return 0;
  }
  if (sub) {
    sub->S = S;
    sub->t0 = t0;
    sub->t1 = t1;
    sub->e0 = c0 >= 0 ? -1 : e0;
    sub->e1 = c1 >= 0 ? -1 : e1;
    sub->c0 = c0;
    sub->c1 = c1;
  }
  return 1;
}
// Whether an uncut grid triangle lies in the foreground: by a
// segment along an edge (side), a corner off the polyline, else its centroid.
__device__ __forceinline__ int pre_uncut_side(const Img& d, const Geo& g, const double2 (&c)[3], const int32_t (&bnd)[3],
                                              int side, const PreBits& B) {
  if (side >= 0) return side;
  double x = c[0].x, y = c[0].y;
  if (bnd[0] >= 0) {
    const bool one = bnd[1] < 0, two = bnd[2] < 0;
    x = one ? c[1].x : c[2].x;
    y = one ? c[1].y : c[2].y;
    if (!one && !two) {
      x = y = 0.0;
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        x += c[j].x / 3;
        y += c[j].y / 3;
      }
    }
  }
  return pre_inside_point(d, g, x, y, &B);
}

__global__ void __launch_bounds__(256, 4) k_pre_mesh_probe_plain(OneSrc src, PreArgs P, Shared sh) {
  const Img& d = src.d;
  const Geo g = d.g;
  const int64_t T = sh.seg_off[sh.nseg].x;  // touched owners
  for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < T; t += (int64_t)gridDim.x * 256) {
    int k, i;
    pre_tl_owner(g, P, t, k, i);
    const int o = k & 1;
    const int64_t v = (int64_t)k * g.NI + i, vd = v + g.NI + o;  // vd: vdr
    const bool whole = pre_slot_ok(g, k, i, 0) && pre_slot_ok(g, k, i, 1);
    const uint32_t fv = P.flags[v], fr = whole ? P.flags[v + 1] : 0u, fdl = whole ? P.flags[vd - 1] : 0u,
                   fdr = whole ? P.flags[vd] : 0u;
    if (!whole || (fv & 7u) || (fdl & 1u) || (fr & 2u)) {  // at the grid's border, or with a split side
      P.rtri[v] = kPreTodo;
      continue;
    }
    const double2 A = pre_place<false>(P, g, v, k, i, fv), Br = pre_place<false>(P, g, v + 1, k, i + 1, fr),
                  Cl = pre_place<false>(P, g, vd - 1, k + 1, i + o - 1, fdl), Dr = pre_place<false>(P, g, vd, k + 1, i + o, fdr);
    const int32_t sv = P.snap_mid[v], sr = P.snap_mid[v + 1], sl = P.snap_mid[vd - 1], sd = P.snap_mid[vd];
    PreBits Bits;
    pre_owner_bits(d, g, P, k, i, Bits);
    const int32_t bv = (fv & kPreSnapped) ? sv : -1, br = (fr & kPreSnapped) ? sr : -1,
                  bl = (fdl & kPreSnapped) ? sl : -1, bd = (fdr & kPreSnapped) ? sd : -1;
    const double2 cb[3] = {A, Dr, Cl}, ca[3] = {A, Br, Dr};
    const int32_t nb[3] = {bv, bd, bl}, na[3] = {bv, br, bd};
    int side_b = -1, side_a = -1, cut_b = 0, cut_a = 0, n0 = 0, n1 = 0, n2 = 0;
    const double m = 1e-9;
    pre_segs_in_box(d, g, fmin(fmin(A.x, Br.x), fmin(Cl.x, Dr.x)) - m, fmax(fmax(A.x, Br.x), fmax(Cl.x, Dr.x)) + m,
                    fmin(fmin(A.y, Br.y), fmin(Cl.y, Dr.y)) - m, fmax(fmax(A.y, Br.y), fmax(Cl.y, Dr.y)) + m,
                    [&](const PreSeg& S) {
      double pb[3], qb[3], pa[3], qa[3], p1, q1;
      pre_half(S, A, Dr, bv, bd, pb[0], qb[0]);
      pre_half(S, Dr, Cl, bd, bl, pb[1], qb[1]);
      pre_half(S, Cl, A, bl, bv, pb[2], qb[2]);
      pre_half(S, A, Br, bv, br, pa[0], qa[0]);
      pre_half(S, Br, Dr, br, bd, pa[1], qa[1]);
      pre_half(S, Dr, A, bd, bv, pa[2], qa[2]);
      pre_half(S, A, Cl, bv, bl, p1, q1);
      cut_b |= pre_clip(S, cb, nb, pb, qb, side_b);
      cut_a |= pre_clip(S, ca, na, pa, qa, side_a);
      // crossings of E0 = A Br, E1 = A Cl, E2 = A Dr at an interior point of both
      const double hx = S.qx - S.px, hy = S.qy - S.py;
      const double ev = hx * (A.y - S.py) - hy * (A.x - S.px);
      auto crosses = [&](double p, double q, double2 W) {
        const double ew = hx * (W.y - S.py) - hy * (W.x - S.px);
        return (int)(((p > 0.0 && q < 0.0) || (p < 0.0 && q > 0.0)) && ((ev > 0.0 && ew < 0.0) || (ev < 0.0 && ew > 0.0)));
      };
      n0 += crosses(pa[0], qa[0], Br);
      n1 += crosses(p1, q1, Cl);
      n2 += crosses(pb[0], qb[0], Dr);
    }, &Bits);
    if (n0 > 3 || n1 > 3 || n2 > 3) pre_error(P);  // more crossings of one grid edge than the numbering holds
    uint32_t rt = ((uint32_t)cut_b << 28) | ((uint32_t)cut_a << 30);
    uint32_t rc = kPrePlain | (uint32_t)min(n0, 3) | ((uint32_t)min(n1, 3) << 4) | ((uint32_t)min(n2, 3) << 8);
    const bool in_b = !cut_b && pre_uncut_side(d, g, cb, nb, side_b, Bits);
    const bool in_a = !cut_a && pre_uncut_side(d, g, ca, na, side_a, Bits);
    if (in_b) {
      rt |= 1u;
      rc += 1u << 19;
      P.used[vd - 1] = 1;
    }
    if (in_a) {
      rt |= 1u << 12;
      rc += 1u << 19;
      P.used[v + 1] = 1;
    }
    if (in_a || in_b) {
      P.used[v] = 1;
      P.used[vd] = 1;
    }
    P.rtri[v] = rt;
    P.rcount[v] = rc;
  }
}

// The owners marked kPreTodo, 64 at a time: a lane per grid triangle, then a
// lane per edge slot in two rounds, their results added up in LDS.  A lane that
// goes through an owner's four triangles and eight edges waits for twelve
// chains of loads in turn: 95 us for the few owners of a 1024 x 1024 image, where
// this takes 38 (8192 x 8192: 521).
constexpr int kPreOwners = 64;
__global__ void __launch_bounds__(256) k_pre_mesh_probe_owner(OneSrc src, PreArgs P, Shared sh) {
  __shared__ int32_t dl[256 + kPreOwners];
  __shared__ uint32_t rt[kPreOwners], rc[kPreOwners];
  __shared__ int nd;
  const Img& d = src.d;
  const Geo g = d.g;
  if (threadIdx.x == 0) nd = 0;
  __syncthreads();
  const int64_t T = sh.seg_off[sh.nseg].x;
  for (int64_t base = (int64_t)blockIdx.x * 256;; base += (int64_t)gridDim.x * 256) {
    const bool more = base < T;  // uniform
    const int64_t it = base + threadIdx.x;
    if (more && it < T) {
      const int32_t v = P.tlist[it];
      if (P.rtri[v] == kPreTodo) dl[atomicAdd(&nd, 1)] = v;
    }
    __syncthreads();
    int m = nd;
    while (m >= kPreOwners || (!more && m > 0)) {  // uniform
      const int take = min(m, kPreOwners);
      const int32_t* const own = dl + (m - take);
      if (threadIdx.x < kPreOwners) rt[threadIdx.x] = rc[threadIdx.x] = 0u;
      __syncthreads();
      for (int r = 0; r < 3; ++r) {
        const int q = r == 0 ? (int)threadIdx.x >> 2 : (((r - 1) * 256 + (int)threadIdx.x) >> 3);
        if (q >= take) continue;
        const uint32_t v = (uint32_t)own[q];
        const int kk = (int)(v / (uint32_t)g.NI), ii = (int)(v - (uint32_t)kk * (uint32_t)g.NI);
        const PreSlots S = pre_owner_slots(P, g, kk, ii);
        PreBits Bits;
        pre_owner_bits(d, g, P, kk, ii, Bits);
        if (r == 0) {
          const int z = (int)threadIdx.x & 3;
          PreGT Tg;
          if (!pre_owner_tri(P, g, kk, ii, S, z, Tg)) continue;
          const double2 c[3] = {make_double2(Tg.c[0].x, Tg.c[0].y), make_double2(Tg.c[1].x, Tg.c[1].y),
                                make_double2(Tg.c[2].x, Tg.c[2].y)};
          const int32_t bnd[3] = {Tg.c[0].bnd, Tg.c[1].bnd, Tg.c[2].bnd};
          int cut = 0, side = -1;
          const double m = 1e-9;
          pre_segs_in_box(d, g, fmin(c[0].x, fmin(c[1].x, c[2].x)) - m, fmax(c[0].x, fmax(c[1].x, c[2].x)) + m,
                          fmin(c[0].y, fmin(c[1].y, c[2].y)) - m, fmax(c[0].y, fmax(c[1].y, c[2].y)) + m,
                          [&](const PreSeg& Sg) {
            double fp[3], fq[3];
#pragma unroll
            for (int e = 0; e < 3; ++e) pre_half(Sg, c[e], c[(e + 1) % 3], bnd[e], bnd[(e + 1) % 3], fp[e], fq[e]);
            cut |= pre_clip(Sg, c, bnd, fp, fq, side);
          }, &Bits);
          if (cut) {  // the cut triangles' pass takes it
            atomicOr(&rt[q], 1u << (28 + z));
          } else if (pre_uncut_side(d, g, c, bnd, side, Bits)) {
#pragma unroll
            for (int j = 0; j < 3; ++j) P.used[Tg.c[j].id] = 1;
            atomicOr(&rt[q], 1u << (6 * z));
            atomicAdd(&rc[q], 1u << 19);
          }
        } else {
          const int e = (int)threadIdx.x & 7;
          PreGV A, B;
          if (!pre_edge_slot(P, g, kk, ii, S, e, A, B)) continue;
          int c = 0;
          pre_edge_crossings(d, g, A, B, [&](const PreSeg&, double) { ++c; }, &Bits);
          if (c > 3) {  // more crossings of one grid edge than the numbering holds
            pre_error(P);
            c = 3;
          }
          atomicAdd(&rc[q], (uint32_t)c << (2 * e));
        }
      }
      __syncthreads();
      if ((int)threadIdx.x < take) {
        P.rtri[own[threadIdx.x]] = rt[threadIdx.x];
        P.rcount[own[threadIdx.x]] = rc[threadIdx.x];
      }
      m -= take;
      __syncthreads();
    }
    if (threadIdx.x == 0) nd = m;
    __syncthreads();
    if (!more) break;
  }
}

// Exclusive scan in place of nblk block counts by one block of 1024; *total
// receives their sum.
__device__ __forceinline__ void pre_scan_blocks(int64_t* a, int64_t nblk, int64_t* total) {
  __shared__ int64_t part[16];
  int64_t run = 0;
  for (int64_t b = 0; b < nblk; b += 1024) {
    const int64_t j = b + threadIdx.x;
    const int64_t x = j < nblk ? a[j] : 0;
    // block-wide exclusive scan of 1024 int64 values (sixteen waves of 64)
    int64_t incl = x;
    for (int off = 1; off < 64; off <<= 1) {
      const int64_t y = __shfl_up(incl, off);
      if ((int)(threadIdx.x & 63) >= off) incl += y;
    }
    if ((threadIdx.x & 63) == 63) part[threadIdx.x >> 6] = incl;
    __syncthreads();
    int64_t before = run;
    for (int w = 0; w < 16; ++w) {
      const int64_t p = part[w];
      before += w < (int)(threadIdx.x >> 6) ? p : 0;
      run += p;
    }
    if (j < nblk) a[j] = before + incl - x;
    __syncthreads();
  }
  if (threadIdx.x == 0) *total = run;
}
// Slots of the cut grid triangles, kPreCScan list positions to a block: the
// block's triangles take a run of slots with one atomic (which run does not
// matter: a slot is only a place to keep a triangle's output), and each
// position its first one (clamped to 32 bits: slots past the room keep
// nothing).
constexpr int kPreCScan = 2048;
__global__ void __launch_bounds__(256) k_pre_cut_slots(PreArgs P, Shared sh) {
  __shared__ int part[4];
  __shared__ int64_t base;
  const int64_t T = sh.seg_off[sh.nseg].x;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  constexpr int kPer = kPreCScan / 256;
  for (int64_t b0 = (int64_t)blockIdx.x * kPreCScan; b0 < T; b0 += (int64_t)gridDim.x * kPreCScan) {
    uint32_t cuts[kPer];
    int n = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int64_t t = b0 + q * 256 + threadIdx.x;
      cuts[q] = t < T ? P.rtri[P.tlist[t]] >> 28 : 0u;
      n += __builtin_popcount(cuts[q]);
    }
    const int incl = wave_incl_scan_dpp(n);
    if (lane == 63) part[wv] = incl;
    __syncthreads();
    if (threadIdx.x == 0)
      base = (int64_t)atomicAdd((unsigned long long*)&P.counts[4], (unsigned long long)(part[0] + part[1] + part[2] + part[3]));
    __syncthreads();
    int64_t slot = base + incl - n;
    for (int w = 0; w < wv; ++w) slot += part[w];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int64_t t = b0 + q * 256 + threadIdx.x;
      if (t < T) P.cbase[t] = (int32_t)min(slot, (int64_t)0x7fffffff);
      for (uint32_t c = cuts[q]; c; c &= c - 1, ++slot)
        if (slot < P.ccap) P.citem[slot] = 4 * (uint64_t)t + __builtin_ctz(c);
    }
    __syncthreads();
  }
}

// A cut grid triangle subdivided, on point numbers of three bits in packed words (the
// boundary cycle, the faces) and the points' places in LDS: points, pieces and faces
// in local arrays took 0.9 KB of scratch memory a lane and moved 3.5 GB through
// memory for 2.3 M triangles (1.70 ms on the 8192 x 8192 image; this 0.44 ms).
struct PreCutWork {
  uint32_t head, ends, tri[2];  // as in PreCut
  int32_t id[3], eo[3];
  uint32_t corners;  // those that an output triangle uses
  int nt;            // output triangles
  uint32_t crossed;  // ends that are crossings; bit 4: a vertex inside
};
// Triangle z of owner (kk, ii): its output to K, the places of crossing k and of
// the vertex inside to pt[3 + k] and pt[7] at threadIdx.x.  false: there is no such
// triangle.  After an error (raised) K is empty.
__device__ __forceinline__ bool pre_cut_subdivide(const Img& d, const Geo& g, const PreArgs& P, int kk, int ii, int z,
                                                  double2 (*pt)[256], PreCutWork& K) {
  K.head = K.ends = K.tri[0] = K.tri[1] = K.corners = K.crossed = 0u;
  K.nt = 0;
  const PreSlots S = pre_owner_slots(P, g, kk, ii);
  PreBits Bits;
  pre_owner_bits(d, g, P, kk, ii, Bits);
  PreGT T;
  if (!pre_owner_tri(P, g, kk, ii, S, z, T)) return false;  // (a cut bit is set for triangles that are there only)
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    K.id[j] = T.c[j].id;
    K.eo[j] = T.eo[j];
  }
  const double2 c[3] = {make_double2(T.c[0].x, T.c[0].y), make_double2(T.c[1].x, T.c[1].y), make_double2(T.c[2].x, T.c[2].y)};
  const int32_t bnd[3] = {T.c[0].bnd, T.c[1].bnd, T.c[2].bnd};
  // 1. the segments inside, clipped
  PreSub s0, s1;
  int nsub = 0;
  const double m = 1e-9;
  pre_segs_in_box(d, g, fmin(c[0].x, fmin(c[1].x, c[2].x)) - m, fmax(c[0].x, fmax(c[1].x, c[2].x)) + m,
                  fmin(c[0].y, fmin(c[1].y, c[2].y)) - m, fmax(c[0].y, fmax(c[1].y, c[2].y)) + m, [&](const PreSeg& Sg) {
    double fp[3], fq[3];
#pragma unroll
    for (int e = 0; e < 3; ++e) pre_half(Sg, c[e], c[(e + 1) % 3], bnd[e], bnd[(e + 1) % 3], fp[e], fq[e]);
    PreSub sb;
    int side = -1;
    if (!pre_clip(Sg, c, bnd, fp, fq, side, &sb)) return;
    if (nsub == 0) s0 = sb;
    if (nsub == 1) s1 = sb;
    ++nsub;
  }, &Bits);
  bool bad = nsub < 1 || nsub > 2;
  if (nsub == 2) {  // chain order
    if (s1.S.jq == s0.S.jp) {
      const PreSub x = s0;
      s0 = s1;
      s1 = x;
    }
    bad = bad || s0.S.jq != s1.S.jp;
  }
  // 2. the pieces' ends: a corner, a crossing of an edge, or (between the two
  // segments of one piece) the polyline vertex inside
  const bool in0 = s0.c1 < 0 && s0.e1 < 0, in1 = nsub == 2 && s1.c0 < 0 && s1.e0 < 0;
  const bool one = nsub == 1 || in0;  // one piece
  const bool inner = nsub == 2 && in0;
  bad = bad || (s0.c0 < 0 && s0.e0 < 0) || (nsub == 1 ? in0 : (in0 != in1 || (s1.c1 < 0 && s1.e1 < 0)));
  if (bad) {  // more than two segments, or a piece that does not join or ends inside
    pre_error(P);
    return true;
  }
  const PreSeg& sl = inner ? s1.S : s0.S;  // of end 1
  const int ec[4] = {s0.c0, inner ? s1.c1 : s0.c1, one ? -1 : s1.c0, one ? -1 : s1.c1};
  const int ee[4] = {s0.c0 >= 0 ? -1 : s0.e0, inner ? (s1.c1 >= 0 ? -1 : s1.e1) : (s0.c1 >= 0 ? -1 : s0.e1),
                     one || s1.c0 >= 0 ? -1 : s1.e0, one || s1.c1 >= 0 ? -1 : s1.e1};
#pragma unroll
  for (int j = 0; j < 3; ++j) pt[j][threadIdx.x] = c[j];
  if (inner) pt[7][threadIdx.x] = make_double2(s0.S.qx, s0.S.qy);
  double te[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    te[k] = 0.0;
    if (ee[k] < 0) continue;
    const PreSeg& Sg = k == 0 ? s0.S : (k == 1 ? sl : s1.S);
    const PreGV A = pre_sel3(T.c[0], T.c[1], T.c[2], ee[k]);
    const PreGV B = pre_sel3(T.c[1], T.c[2], T.c[0], ee[k]);
    double2 q;
    pre_crossing_xy(Sg, A.id < B.id ? A : B, A.id < B.id ? B : A, q.x, q.y);
    pt[3 + k][threadIdx.x] = q;
    const double L2 = (B.x - A.x) * (B.x - A.x) + (B.y - A.y) * (B.y - A.y);
    te[k] = ((q.x - A.x) * (B.x - A.x) + (q.y - A.y) * (B.y - A.y)) / L2;
    bad = bad || !(te[k] > 0 && te[k] < 1);
  }
  // 3. the boundary cycle: the corners and the crossings on each edge in order;
  // nibble x of cyc: the point at place x, of cend: the end that sits there + 1,
  // nibble k of place: where end k sits
  uint32_t cyc = 0, cend = 0, place = 0, ends = 0;
  int on[3] = {0, 0, 0};  // crossings per edge
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int e = 0; e < 3; ++e) on[e] += ee[k] == e;
  const int first[3] = {0, 1 + on[0], 2 + on[0] + on[1]};  // place of corner e
#pragma unroll
  for (int j = 0; j < 3; ++j) cyc |= (uint32_t)j << (4 * first[j]);
  const int n = 3 + on[0] + on[1] + on[2];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (ee[k] < 0 && ec[k] < 0) continue;
    int at;
    if (ec[k] >= 0) {
      at = pre_sel3(first[0], first[1], first[2], ec[k]);
      bad = bad || ((cend >> (4 * at)) & 15u) != 0u;  // two pieces at one corner
    } else {
      int rank = 0;
#pragma unroll
      for (int o = 0; o < 4; ++o) rank += o != k && ee[o] == ee[k] && (te[o] < te[k] || (te[o] == te[k] && o < k));
      const int cnt = pre_sel3(on[0], on[1], on[2], ee[k]);
      at = pre_sel3(first[0], first[1], first[2], ee[k]) + 1 + rank;
      cyc |= (uint32_t)(3 + k) << (4 * at);
      const int32_t ia = pre_sel3(T.c[0].id, T.c[1].id, T.c[2].id, ee[k]), ib = pre_sel3(T.c[1].id, T.c[2].id, T.c[0].id, ee[k]);
      ends |= (0x80u | (uint32_t)ee[k] | ((uint32_t)(ia < ib ? rank : cnt - 1 - rank) << 2)) << (8 * k);
    }
    cend |= (uint32_t)(k + 1) << (4 * at);
    place |= (uint32_t)at << (4 * k);
  }
  // 4. faces: walk the cycle; at a piece end reached along the boundary, follow
  // the piece; the foreground ones by the template rule
  uint32_t used = 0;
  int nt = 0;
  for (int st = 0; st < n && !bad; ++st) {
    if ((used >> st) & 1u) continue;
    uint64_t face = 0;  // nibble j: point j of the face
    int fm = 0, side = -1, at = st;
    for (int guard = 0; guard < 16; ++guard) {
      if ((used >> at) & 1u) break;
      used |= 1u << at;
      face |= (uint64_t)((cyc >> (4 * at)) & 15u) << (4 * fm);
      ++fm;
      const int nx = at + 1 == n ? 0 : at + 1;
      const int k = (int)((cend >> (4 * nx)) & 15u) - 1;
      if (k >= 0) {
        const int s2 = (k & 1) ? 0 : 1;
        if (side >= 0 && side != s2) bad = true;  // a face on both sides of the chain
        side = s2;
        face |= (uint64_t)((cyc >> (4 * nx)) & 15u) << (4 * fm);
        ++fm;
        if (inner) {
          face |= 7ull << (4 * fm);
          ++fm;
        }
        at = (int)((place >> (4 * (k ^ 1))) & 15u);
      } else {
        at = nx;
      }
      if (at == st || fm > 12) break;
    }
    if (side != 1 || bad) continue;
    if (fm < 3) {  // degenerate face
      bad = true;
      continue;
    }
    int apex = -1, low = 8;
    bool has_corner = false;
    for (int j = 0; j < fm; ++j) {
      const int q = (int)(face >> (4 * j)) & 15;
      has_corner = has_corner || q < 3;
      // the earliest chain point: the lowest end; the inner vertex before all
      int o = q == 7 ? -1 : q - 3;
      if (q < 3) {
        const int w = (int)((cend >> (4 * pre_sel3(first[0], first[1], first[2], q))) & 15u);
        o = w ? w - 1 : 8;
      }
      if (o < low) {
        low = o;
        apex = j;
      }
    }
    if (!inner && fm == 4 && !one && !has_corner) {
      // the middle quadrilateral between two chords: diagonal joining their exits
      apex = -1;
      for (int j = 0; j < 4; ++j)
        if (((face >> (4 * j)) & 15u) == 4u) apex = j;
      if (apex < 0 || ((face >> (4 * ((apex + 2) & 3))) & 15u) != 6u) bad = true;  // nested exits not opposite
    }
    if (apex < 0) bad = true;
    if (bad) continue;
    const int pa = (int)(face >> (4 * apex)) & 15;
    const double2 a = pt[pa][threadIdx.x];
    for (int j = 1; j + 1 < fm; ++j) {
      const int jb = apex + j >= fm ? apex + j - fm : apex + j, jc = jb + 1 == fm ? 0 : jb + 1;
      const int pb = (int)(face >> (4 * jb)) & 15, pc = (int)(face >> (4 * jc)) & 15;
      const double2 b = pt[pb][threadIdx.x], e = pt[pc][threadIdx.x];
      if (!((b.x - a.x) * (e.y - a.y) - (b.y - a.y) * (e.x - a.x) > 0.0)) pre_error(P);
      const uint32_t w = (uint32_t)(pa | (pb << 3) | (pc << 6)) << (9 * (nt & 1));
      K.tri[0] |= nt < 2 ? w : 0u;
      K.tri[1] |= nt >= 2 && nt < kPreKeep ? w : 0u;
      K.corners |= (1u << pa) | (1u << pb) | (1u << pc);
      ++nt;
    }
  }
  if (bad || nt > kPreKeep) {
    pre_error(P);
    K.tri[0] = K.tri[1] = K.corners = 0u;
    return true;
  }
  K.nt = nt;
  K.head = (uint32_t)nt | ((uint32_t)T.es[0] << 8) | ((uint32_t)T.es[1] << 12) | ((uint32_t)T.es[2] << 16) |
           (inner ? 1u << 20 : 0u);
  K.ends = ends;
#pragma unroll
  for (int k = 0; k < 4; ++k) K.crossed |= ee[k] >= 0 ? 1u << k : 0u;
  if (inner) K.crossed |= 16u;
  return true;
}
// Its counts, and the corners it uses.
__device__ __forceinline__ void pre_cut_counted(const PreArgs& P, int64_t v, int z, const PreCutWork& K) {
#pragma unroll
  for (int j = 0; j < 3; ++j)
    if ((K.corners >> j) & 1u) P.used[K.id[j]] = 1;
  pre_add_counts(P, v, z, K.nt, (int)(K.crossed >> 4));
}
// The cut grid triangles that have a slot, one lane each.  Their triangles are kept
// for k_pre_cut_write, with the crossings' edges, order and places.
__global__ void __launch_bounds__(256, 3) k_pre_cut_make(OneSrc src, PreArgs P) {
  __shared__ double2 pt[8][256];
  const Img& d = src.d;
  const Geo g = d.g;
  const int64_t n_items = min(P.counts[4], P.ccap);
  for (int64_t slot = (int64_t)blockIdx.x * 256 + threadIdx.x; slot < n_items; slot += (int64_t)gridDim.x * 256) {
    const uint64_t item = P.citem[slot];
    const int z = (int)(item & 3u);
    int kk, ii;
    pre_tl_owner(g, P, (int64_t)(item >> 2), kk, ii);
    PreCutWork W;
    const bool there = pre_cut_subdivide(d, g, P, kk, ii, z, pt, W);
    if (there) pre_cut_counted(P, (int64_t)kk * g.NI + ii, z, W);
    PreCut& K = P.cstore[slot];
    K.head = W.head;
    K.ends = W.ends;
    if (W.head == 0u) continue;  // nothing to write
    K.tri[0] = W.tri[0];
    K.tri[1] = W.tri[1];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      K.id[j] = W.id[j];
      K.eo[j] = W.eo[j];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if ((W.crossed >> k) & 1u) K.pos[k] = pt[3 + k][threadIdx.x];
    if (W.crossed & 16u) K.pos[4] = pt[7][threadIdx.x];
  }
}

// The cut grid triangles beyond the slots, gathered per block and counted on full
// blocks; nothing of them is kept (k_pre_mesh_cut_rest subdivides them again).
// There are none on smooth shapes, where the room, one for every sixteen owners,
// does; on noise of one to three pixels most have no slot.
__global__ void __launch_bounds__(256, 3) k_pre_mesh_cut_count(OneSrc src, PreArgs P, Shared sh) {
  __shared__ double2 pt[8][256];
  __shared__ int64_t dl[512];
  __shared__ int nd;
  if (P.counts[4] <= P.ccap) return;  // uniform
  const Img& d = src.d;
  const Geo g = d.g;
  if (threadIdx.x == 0) nd = 0;
  __syncthreads();
  const int64_t T = sh.seg_off[sh.nseg].x;
  pre_dense(4 * T, dl, &nd, [&](int64_t it) -> bool {
    const uint32_t rt = P.rtri[P.tlist[it >> 2]];
    return ((rt >> (28 + (it & 3))) & 1u) && pre_cut_slot(P, it >> 2, (int)(it & 3), rt) >= P.ccap;
  }, [&](int64_t it) {
    int kk, ii;
    pre_tl_owner(g, P, it >> 2, kk, ii);
    PreCutWork W;
    if (pre_cut_subdivide(d, g, P, kk, ii, (int)(it & 3), pt, W))
      pre_cut_counted(P, (int64_t)kk * g.NI + ii, (int)(it & 3), W);
  });
}

// What is known of a row segment's owners, every load before the first use: the
// inside and touched bits (uniform), the counts of the touched ones (lane l: owner
// v + 64 j, v that of step 0).
__device__ __forceinline__ void pre_segment_owners(const PreArgs& P, int64_t seg, int64_t v, int lane,
                                                   unsigned long long (&ins)[4], unsigned long long (&tou)[4],
                                                   uint32_t (&rc)[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    ins[j] = P.inside[4 * seg + j];
    tou[j] = pre_touched64(P, seg, j);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) rc[j] = (tou[j] >> lane) & 1ull ? P.rcount[v + 64 * j] : 0u;
}
// Per row segment: new vertices, triangles and cut grid triangles of its
// owners, the input of the scan; counts[3] keeps the number of touched owners.
__global__ void __launch_bounds__(256) k_pre_mesh_segsum(OneSrc src, PreArgs P, Shared sh) {
  const Geo g = src.d.g;
  if (blockIdx.x == 0 && threadIdx.x == 0) P.counts[3] = sh.seg_off[sh.nseg].x;
  int64_t seg;
  int k, i0;
  if (!pre_segment(g, sh, seg, k, i0)) return;  // wave-uniform
  const int lane = threadIdx.x & 63;
  int nv = 0, nt = 0, nc = 0;
  unsigned long long ins[4], tou[4];
  uint32_t rc[4];
  pre_segment_owners(P, seg, (int64_t)k * g.NI + i0 + lane, lane, ins, tou, rc);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int i = i0 + 64 * j + lane;
    if ((ins[j] >> lane) & 1ull) nt += (int)pre_slot_ok(g, k, i, 0) + (int)pre_slot_ok(g, k, i, 1);
    nv += pre_rc_before(rc[j], 8) + pre_rc_inner(rc[j]);
    nt += pre_rc_tris(rc[j]);
    nc += pre_rc_cut(rc[j]);
  }
  nv = __builtin_amdgcn_readlane(wave_incl_scan_dpp(nv), 63);
  nt = __builtin_amdgcn_readlane(wave_incl_scan_dpp(nt), 63);
  nc = __builtin_amdgcn_readlane(wave_incl_scan_dpp(nc), 63);
  if (lane == 0) {
    sh.seg_cnt[seg] = make_int4(nv, nt, nc, 0);
    sh.seg_slow[seg] = 0ull;
  }
}

// Output triangles at their offsets, with their codes: the slots of a quiet owner
// inside, and the uncut ones of a plain touched owner, as they are (code 0).  The
// 64 owners of a wave step hold consecutive output ranges: their triangles are
// staged in LDS by rank and lane j writes ranks j and j + 64 (the other ranks are
// left to the dense passes).  For those each touched owner's first output triangle
// and first new vertex are noted: its crossings, edge slot by edge slot in order
// from the edge's lower-numbered end, then the polyline vertices inside its
// triangles (relative to the grid vertices kept).
// The owners' states are bits and the corners' ids a rank among bits: with a word
// of counts and an id kept per owner and vertex, and the plain owners' uncut
// triangles in a pass over the list, this took 923 us on the 8192 x 8192
// image, together, and now 562 (418 here).
__global__ void __launch_bounds__(256) k_pre_mesh_triangles(OneSrc src, PreArgs P, Shared sh) {
  __shared__ Tri3 stage[4][128];
  __shared__ uint8_t full[4][128];
  const Geo g = src.d.g;
  int64_t seg;
  int k, i0;
  if (!pre_segment(g, sh, seg, k, i0)) return;  // wave-uniform
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const unsigned long long planned = pre_planned(P) ? ~0ull : 0ull;
  const longlong4 off = sh.seg_off[seg];
  const int64_t t0 = off.y;
  int64_t vacc = off.x;
  const int o = k & 1;
  int acc = 0;
  unsigned long long inw[4], tow[4];
  uint32_t rcs[4], rts[4];
  pre_segment_owners(P, seg, (int64_t)k * g.NI + i0 + lane, lane, inw, tow, rcs);
#pragma unroll
  for (int j = 0; j < 4; ++j) rts[j] = rcs[j] & kPrePlain ? P.rtri[(int64_t)k * g.NI + i0 + lane + 64 * j] : 0u;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const unsigned long long ins = inw[j] & planned, tou = tow[j] & planned;
    if ((ins | tou) == 0ull) continue;
    const int i = i0 + 64 * j + lane;
    const int64_t v = (int64_t)k * g.NI + i;
    const bool in = (ins >> lane) & 1ull, touched = (tou >> lane) & 1ull;
    bool tb = in && pre_slot_ok(g, k, i, 0), ta = in && pre_slot_ok(g, k, i, 1);
    const uint32_t rc = rcs[j];
    const int n = in ? (int)tb + (int)ta : pre_rc_tris(rc);
    int nb = (int)tb;  // output triangles of slot Tb
    if (rc & kPrePlain) {
      const uint32_t rt = rts[j];
      nb = (int)(rt & 63u);
      tb = nb && !((rt >> 28) & 1u);
      ta = ((rt >> 12) & 63u) && !((rt >> 30) & 1u);
    }
    const int incl = wave_incl_scan_dpp(n);
    const int tot = __builtin_amdgcn_readlane(incl, 63);  // at most 4 * 64 (a touched owner: 4 * 63)
    if (tou) {
      const int nn = pre_rc_before(rc, 8) + pre_rc_inner(rc), vincl = wave_incl_scan_dpp(nn);
      if (nn) P.rbase[v] = vacc + (vincl - nn);
      vacc += __builtin_amdgcn_readlane(vincl, 63);
      if (touched && n > 0) P.rtbase[v] = t0 + acc + (incl - n);
    }
    // the corners' ids: a kept triangle's corners are all used, so v's right
    // neighbour is the next one, and so it is in the row below
    Tri3 Tb = {}, Ta = {};
    if (tb || ta) {
      const int32_t a = pre_vertex(P, v), dr = pre_vertex(P, v + g.NI + o);
      Tb.a = Ta.a = a;
      Tb.b = Ta.c = dr;
      Tb.c = dr - 1;
      Ta.b = a + 1;
    }
    for (int b = 0; b < tot; b += 128) {  // uniform
      full[wv][lane] = full[wv][lane + 64] = 0;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const int r = incl - n - b, r2 = r + nb;
      if (tb && r >= 0 && r < 128) {
        stage[wv][r] = Tb;
        full[wv][r] = 1;
      }
      if (ta && r2 >= 0 && r2 < 128) {
        stage[wv][r2] = Ta;
        full[wv][r2] = 1;
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int q = lane + 64 * h;
        const int64_t pos = t0 + acc + b + q;
        if (full[wv][q] && pos < P.otcap) {
          *reinterpret_cast<Tri3*>(P.otris + 3 * pos) = stage[wv][q];
          P.ocodes[pos] = 0;
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    acc += tot;
  }
}

// Uncut triangles (in the foreground) of the touched owners that are not plain,
// 64 of these owners at a time, a lane per grid triangle: written as they are.
__global__ void __launch_bounds__(256) k_pre_mesh_whole_tris(OneSrc src, PreArgs P) {
  __shared__ int32_t dl[256 + kPreOwners];
  __shared__ int nd;
  const Geo g = src.d.g;
  if (threadIdx.x == 0) nd = 0;
  __syncthreads();
  int64_t T = P.counts[3];
  if (!pre_planned(P)) T = 0;
  for (int64_t base = (int64_t)blockIdx.x * 256;; base += (int64_t)gridDim.x * 256) {
    const bool more = base < T;  // uniform
    const int64_t it = base + threadIdx.x;
    if (more && it < T) {
      const int32_t v = P.tlist[it];
      const uint32_t rc = P.rcount[v];
      if (!(rc & kPrePlain) && pre_rc_tris(rc)) dl[atomicAdd(&nd, 1)] = v;
    }
    __syncthreads();
    int m = nd;
    while (m >= kPreOwners || (!more && m > 0)) {  // uniform
      const int take = min(m, kPreOwners), z = (int)threadIdx.x & 3;
      if ((int)threadIdx.x < 4 * take) {
        const uint32_t v = (uint32_t)dl[m - take + ((int)threadIdx.x >> 2)];
        const uint32_t rt = P.rtri[v];
        if (((rt >> (6 * z)) & 63u) && !((rt >> (28 + z)) & 1u)) {
          int before = 0;
          for (int z2 = 0; z2 < z; ++z2) before += (int)((rt >> (6 * z2)) & 63u);
          const int64_t pos = P.rtbase[v] + before;
          const int kk = (int)(v / (uint32_t)g.NI), ii = (int)(v - (uint32_t)kk * (uint32_t)g.NI);
          const PreSlots S = pre_owner_slots(P, g, kk, ii);
          PreGT Tg;
          if (pre_owner_tri(P, g, kk, ii, S, z, Tg) && pos < P.otcap) {
            Tri3 t3;
            t3.a = pre_vertex(P, Tg.c[0].id);
            t3.b = pre_vertex(P, Tg.c[1].id);
            t3.c = pre_vertex(P, Tg.c[2].id);
            *reinterpret_cast<Tri3*>(P.otris + 3 * pos) = t3;
            P.ocodes[pos] = 0;
          }
        }
      }
      m -= take;
    }
    __syncthreads();
    if (threadIdx.x == 0) nd = m;
    __syncthreads();
    if (!more) break;
  }
}
// Output of cut grid triangle z of owner v (head, ends, t01, t23, kid, keo as in
// PreCut; place(k) the place of crossing k, 4: of the vertex inside): the crossings'
// and the inner vertex's places go to their mesh vertices (the two triangles of an
// edge write the same places), the triangles to theirs, all by number: a crossing is
// the edge owner's first one of that edge plus its order.
template <class Place>
__device__ __forceinline__ void pre_cut_output(const PreArgs& P, const Geo& g, int64_t NV, int64_t v, int z, uint32_t head,
                                               uint32_t ends, uint32_t t01, uint32_t t23, const int32_t (&kid)[3],
                                               const int32_t (&keo)[3], Place place) {
  double2* const Vout = reinterpret_cast<double2*>(P.overts);
  const int kn = (int)(head & 255u);
  const uint32_t rc = P.rcount[v], rt = P.rtri[v];
  int32_t cid[3];  // corners in the mesh (one that no triangle uses has no number, and none is looked at)
  int64_t id[4];
#pragma unroll
  for (int j = 0; j < 3; ++j) cid[j] = pre_vertex(P, kid[j]);
  int64_t eb[3];
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    int cnt = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) cnt += ((ends >> (8 * k)) & 0x83u) == (0x80u | (uint32_t)e);
    eb[e] = 0;
    if (!cnt) continue;
    const int64_t w = keo[e];
    const int es = (int)((head >> (8 + 4 * e)) & 15u);
    const uint32_t rw = pre_owner_counts(P, g, (uint32_t)w);
    if (pre_rc_cross(rw, es) != cnt) {  // the edge and the triangle see other crossings
      pre_error(P);
      eb[e] = P.ovcap;  // no row: an owner without crossings has no base (rbase is not written there)
      continue;
    }
    eb[e] = NV + P.rbase[w] + pre_rc_before(rw, es);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t x = (ends >> (8 * k)) & 255u;
    id[k] = pre_sel3(eb[0], eb[1], eb[2], (int)(x & 3u)) + ((x >> 2) & 3u);
    if ((x & 0x80u) && id[k] < P.ovcap) Vout[id[k]] = place(k);
  }
  int64_t inner = 0;
  if ((head >> 20) & 1u) {
    inner = NV + P.rbase[v] + pre_rc_before(rc, 8) + __builtin_popcount((rt >> 24) & ((1u << z) - 1u));
    if (inner < P.ovcap) Vout[inner] = place(4);
  }
  int before = 0;
  for (int z2 = 0; z2 < z; ++z2) before += (int)((rt >> (6 * z2)) & 63u);
  const int64_t pos = P.rtbase[v] + before;
  auto num = [&](uint32_t p) -> int32_t {
    const int32_t c = pre_sel3(cid[0], cid[1], cid[2], (int)(p & 3u));
    const int32_t x01 = (int32_t)(p == 3u ? id[0] : id[1]), x23 = (int32_t)(p == 5u ? id[2] : id[3]);
    return p < 3u ? c : (p == 7u ? (int32_t)inner : (p < 5u ? x01 : x23));
  };
  for (int j = 0; j < kn; ++j) {
    if (pos + j >= P.otcap) break;
    const uint32_t w = ((j < 2 ? t01 : t23) >> (9 * (j & 1))) & 511u;
    Tri3 t3;
    t3.a = num(w & 7u);
    t3.b = num((w >> 3) & 7u);
    t3.c = num(w >> 6);
    *reinterpret_cast<Tri3*>(P.otris + 3 * (pos + j)) = t3;
    P.ocodes[pos + j] = 1;
  }
}
// The cut grid triangles kept in their slots, one lane each.
__global__ void __launch_bounds__(256) k_pre_cut_write(OneSrc src, PreArgs P) {
  const Geo g = src.d.g;
  int64_t n = min(P.counts[4], P.ccap);
  const int64_t NV = *P.nused;
  if (!pre_planned(P)) n = 0;
  for (int64_t slot = (int64_t)blockIdx.x * 256 + threadIdx.x; slot < n; slot += (int64_t)gridDim.x * 256) {
    const PreCut& K = P.cstore[slot];
    const uint32_t head = K.head, ends = K.ends;
    const int kn = (int)(head & 255u);
    if (kn == 0 && ends == 0u) continue;
    const uint64_t item = P.citem[slot];
    pre_cut_output(P, g, NV, P.tlist[item >> 2], (int)(item & 3u), head, ends, K.tri[0], K.tri[1], K.id, K.eo,
                   [&](int k) { return K.pos[k]; });
  }
}
// The cut grid triangles beyond the slots, subdivided again.
// 2000 x 2000 noise of one pixel (1.6 M cut triangles, 65536 slots), the whole call:
// with points, pieces and faces in local arrays and the vertices looked for by walks
// and subdivisions of their own 7.2 ms (5.6 before any was kept in full), now 2.3.
__global__ void __launch_bounds__(256, 3) k_pre_mesh_cut_rest(OneSrc src, PreArgs P) {
  __shared__ double2 pt[8][256];
  __shared__ int64_t dl[512];
  __shared__ int nd;
  if (P.counts[4] <= P.ccap || !pre_planned(P)) return;  // uniform
  const Img& d = src.d;
  const Geo g = d.g;
  if (threadIdx.x == 0) nd = 0;
  __syncthreads();
  const int64_t T = P.counts[3];
  const int64_t NV = *P.nused;
  pre_dense(4 * T, dl, &nd, [&](int64_t it) -> bool {
    const uint32_t rt = P.rtri[P.tlist[it >> 2]];
    return ((rt >> (28 + (it & 3))) & 1u) && pre_cut_slot(P, it >> 2, (int)(it & 3), rt) >= P.ccap;
  }, [&](int64_t it) {
    int kk, ii;
    pre_tl_owner(g, P, it >> 2, kk, ii);
    PreCutWork W;
    if (pre_cut_subdivide(d, g, P, kk, ii, (int)(it & 3), pt, W) && W.head)
      pre_cut_output(P, g, NV, (int64_t)kk * g.NI + ii, (int)(it & 3), W.head, W.ends, W.tri[0], W.tri[1], W.id, W.eo,
                     [&](int k) { return pt[k == 4 ? 7 : 3 + k][threadIdx.x]; });
  });
}

// Compaction of the grid vertices: the used ones keep their order.  A thread packs
// 64 flags into a word with its rank in its block of kPreVScan vertices (of the NV
// the grid phase made), one block scans the blocks' counts, and the used vertices
// are copied into the mesh, 64 a wave step.  An id is looked up as a rank
// (pre_vertex), so that no pass has to write one per vertex or to go through a
// block's vertices in order (8192 x 8192: 375 -> 240 us; 1024 x 1024, where 74
// blocks had to do all of it, 34 -> 6 us).
__global__ void __launch_bounds__(256) k_pre_vscan_count(PreArgs P) {
  __shared__ int part[4];
  static_assert(kPreVScan == 64 * 256, "a word per thread");
  const int64_t NV = P.gsizes[0] < P.usedcap ? P.gsizes[0] : P.usedcap;
  const int64_t v0 = (int64_t)blockIdx.x * kPreVScan + 64 * (int64_t)threadIdx.x;
  uint64_t bits = 0;
  if (v0 < NV) {  // the flags' region ends on a multiple of 256 bytes
    const uint4* u = reinterpret_cast<const uint4*>(P.used + v0);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint4 x = u[q];
      bits |= (uint64_t)(nz8(x.x, x.y) | (nz8(x.z, x.w) << 8)) << (16 * q);
    }
    if (NV - v0 < 64) bits &= (1ull << (NV - v0)) - 1ull;
  }
  const int n = (int)__popcll(bits), incl = wave_incl_scan_dpp(n), wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 63) part[wv] = incl;
  __syncthreads();
  int before = incl - n;
  for (int w = 0; w < wv; ++w) before += part[w];
  if (v0 < NV) P.uword[v0 >> 6] = PreUsed{bits, before, 0};
  if (threadIdx.x == 255) P.vbsum[blockIdx.x] = before + n;
}
// The mesh's vertices may be numbered, and no pass before this one saw an error.
__device__ __forceinline__ int64_t pre_mesh_status(const PreArgs& P, const Shared& sh) {
  if (*P.nused + sh.seg_off[sh.nseg].x > 0x7fffffffLL) return SBMT_E_INDEX_OVERFLOW;
  if (P.gsizes[5] != SBMT_OK && P.gsizes[5] != SBMT_E_CAPACITY) return P.gsizes[5];  // (no room for triangles is meant there)
  return P.counts[2] ? SBMT_E_PROTOCOL : SBMT_OK;
}
__global__ void __launch_bounds__(1024) k_pre_vscan_top(PreArgs P, Shared sh, int64_t nblk) {
  pre_scan_blocks(P.vbsum, nblk, P.nused);
  if (threadIdx.x == 0 && pre_mesh_status(P, sh) == SBMT_OK)
    for (int q = 0; q < kPreStamp; ++q) P.stamp_at[q] = P.stamp[q];
}
__global__ void __launch_bounds__(256) k_pre_vscan_apply(OneSrc src, PreArgs P) {
  const Geo g = src.d.g;
  const int64_t nlat = (int64_t)g.NK * g.NI;
  int64_t NV = P.gsizes[0] < P.usedcap ? P.gsizes[0] : P.usedcap;
  if (!pre_planned(P)) NV = 0;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr int kPer = kPreApplyWords / 4;
  const int64_t w0 = (int64_t)blockIdx.x * kPreApplyWords + wv * kPer;
  if (64 * w0 >= NV) return;
  const double2* G = reinterpret_cast<const double2*>(P.verts);
  double2* O = reinterpret_cast<double2*>(P.overts);
  const int64_t before = P.vbsum[w0 / (kPreVScan / 64)];  // a block's words lie in one block of the scan
  uint32_t k = (uint32_t)(64 * w0 + lane) / (uint32_t)g.NI, i = (uint32_t)(64 * w0 + lane) - k * (uint32_t)g.NI;
  PreUsed u[kPer];
  uint32_t f[kPer];
#pragma unroll
  for (int q = 0; q < kPer; ++q) {  // every load first
    const int64_t v = 64 * (w0 + q) + lane;
    u[q] = P.uword[64 * (w0 + q) < NV ? w0 + q : w0];
    f[q] = v < nlat ? P.flags[v] : kPreMoved;
  }
  double2 m[kPer];
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int64_t v = 64 * (w0 + q) + lane;
    m[q] = G[v < NV && (f[q] & kPreMoved) ? v : 0];
  }
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int64_t id = before + u[q].base + lanes_below(u[q].bits);
    const double x = lat_x(g, pre_lat_X(g, (int)k, (int)i)), y = lat_y(g, (int)k);
    const bool moved = (f[q] & kPreMoved) != 0;
    if (64 * (w0 + q) < NV && ((u[q].bits >> lane) & 1ull) && id < P.ovcap)
      O[id] = make_double2(moved ? m[q].x : x, moved ? m[q].y : y);
    for (i += 64u; i >= (uint32_t)g.NI; i -= (uint32_t)g.NI) ++k;
  }
}

// The call's counts and status.  fill: a call that did not plan has counts only
// where the workspace holds its plan.
__global__ void k_pre_mesh_sizes(PreArgs P, Shared sh, int64_t* out, bool fill) {
  if (fill && !pre_planned(P)) {
    for (int q = 0; q < 8; ++q) out[q] = 0;
    out[5] = SBMT_E_INVALID_ARG;
    return;
  }
  const longlong4 tot = sh.seg_off[sh.nseg];
  const int64_t NV = *P.nused;
  out[0] = NV + tot.x;        // vertices
  out[1] = tot.y;             // triangles
  out[2] = P.gsizes[2];       // snapped
  out[3] = P.gsizes[3];       // repelled
  out[4] = P.gsizes[4];       // inserted
  out[6] = NV;                // grid vertices in the mesh
  out[7] = tot.z;             // cut grid triangles
  const int64_t st = pre_mesh_status(P, sh);
  out[5] = st == SBMT_OK && (out[0] > P.ovcap || out[1] > P.otcap) ? SBMT_E_CAPACITY : st;
}

// Workspace of the preprocessing: the meshing layout of the image, then the
// per-midpoint words, the per-owner split sides, flags and first inserted
// indices, and the counters and sizes.
struct PreLayout {
  CallLayout L;
  size_t off_mid, off_split, off_flags, off_ins, off_counts, off_out, off_snap, total;
  // the retriangulation (sbmt_preprocess_mesh): per-owner counts and bases, sizes
  size_t off_rcount, off_rtri, off_rbase, off_out2, off_gverts, off_used, off_uword, off_inside, off_vbsum, off_nused,
      off_tlist, off_rtbase, off_cbase, off_citem, off_cstore, off_touched;
  int64_t ccap;      // cut triangles whose output is kept
  int64_t ntouched;  // words of the touched bits
  int64_t nvblk;  // blocks of the vertex compaction scan
  int64_t nmid, nown;
};
static sbmt_status pre_layout(const sbmt_image* img, bool need_ptr, PreLayout* P, bool mesh = false) {
  sbmt_status st = make_call_layout(img, 1, 0, need_ptr, &P->L);
  if (st != SBMT_OK) return st;
  const Geo& g = P->L.g[0];
  P->nmid = 2LL * (g.CH + 2) * (g.CW + 2);
  P->nown = (int64_t)g.NK * g.NI;
  if (P->nmid >= (1LL << 31)) return SBMT_E_INVALID_ARG;  // midpoint ids are int32
  size_t off = align256(P->L.total);
  P->off_mid = off;
  off = align256(off + (size_t)P->nmid);
  P->off_split = off;
  off = align256(off + (size_t)P->nown * 12);
  P->off_flags = off;
  off = align256(off + (size_t)P->nown);
  P->off_ins = off;
  off = align256(off + (size_t)P->nown * 8);
  P->off_counts = off;
  off = align256(off + kPreCounts * 8);
  P->off_out = off;
  off = align256(off + 8 * 8);
  P->off_snap = off;
  off = align256(off + (size_t)P->nown * 4);
  P->off_rcount = P->off_rtri = P->off_rbase = P->off_out2 = 0;
  P->off_gverts = P->off_used = P->off_uword = P->off_inside = P->off_vbsum = P->off_nused = P->off_tlist = P->off_rtbase = 0;
  P->off_cbase = P->off_citem = P->off_cstore = P->off_touched = 0;
  P->ccap = P->ntouched = 0;
  P->nvblk = 0;
  if (mesh) {
    P->off_rcount = off;
    off = align256(off + (size_t)P->nown * 4);
    P->off_rtri = off;
    off = align256(off + (size_t)P->nown * 4);
    P->off_rbase = off;
    off = align256(off + (size_t)P->nown * 8);
    P->off_out2 = off;
    off = align256(off + 8 * 8);
    const int64_t ng = P->nown + P->nmid;  // bound on the grid vertices
    P->nvblk = (ng + kPreVScan - 1) / kPreVScan;
    P->off_gverts = off;
    off = align256(off + (size_t)ng * 16);
    P->off_used = off;
    off = align256(off + (size_t)ng);  // read 64 bytes at a time
    P->off_uword = off;
    off = align256(off + (size_t)((ng + 63) / 64) * sizeof(PreUsed));
    P->off_inside = off;
    off = align256(off + (size_t)(4LL * g.NK * g.NCB) * 8);
    P->off_vbsum = off;
    off = align256(off + (size_t)P->nvblk * 8);
    P->off_nused = off;
    off = align256(off + 8);
    P->off_tlist = off;
    off = align256(off + (size_t)P->nown * 4);
    P->off_rtbase = off;
    off = align256(off + (size_t)P->nown * 8);
    // kept outputs of the cut grid triangles (136 bytes each): room for one in 16
    // owners, in images of few owners for more, but not beyond their base triangles
    P->ntouched = 8LL * g.NK * g.NCB;
    P->off_touched = off;
    off = align256(off + (size_t)P->ntouched * 4);
    P->ccap = std::min<int64_t>(2 * P->nown, std::max<int64_t>(65536, P->nown / 16));
    P->off_cbase = off;
    off = align256(off + (size_t)P->nown * 4);
    P->off_citem = off;
    off = align256(off + (size_t)P->ccap * 8);
    P->off_cstore = off;
    off = align256(off + (size_t)P->ccap * sizeof(PreCut));
  }
  P->total = off;
  return SBMT_OK;
}
// Words a wave enumerates the polyline from (log2): full waves of items where
// there are words enough for four waves per SIMD, else fewer words, down to
// four, so that the waves of a small image run side by side and not their items
// one after the other (Step 3 on 4000 x 3000 with 64 words a wave, 1.5 blocks
// per CU: 106 us; with 16: 45 us).
static int pre_wave_words(const Geo& g) {
  const int64_t words = (int64_t)(g.CH + 1) * g.wpr;
  int shift = 2;
  while (shift < 6 && (words >> (shift + 1)) >= 4096) ++shift;
  return shift;
}
static int64_t pre_word_blocks(const Geo& g) {
  const int64_t per = 4LL << pre_wave_words(g);
  return ((int64_t)(g.CH + 1) * g.wpr + per - 1) / per;
}
static bool pre_thresholds_ok(double a, double b, double c, double h) {
  if (!(a >= 0 && b >= 0 && c >= 0)) return false;
  if (a == 0 && b == 0 && c == 0) return true;
  return b < a / 2 && c * c < a * a / 2 && a < h / 2;
}
