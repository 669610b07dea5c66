// Cotangent Laplacian assembly and explicit heat steps on gfx950 (linear
// finite elements on an SBMT mesh; the diffusion setting of App. H).
//
// Assembly:
//   1. every vertex's incident triangles in eight slots of its own (32 bytes),
//      from one pass over the triangles (k_incident); the few vertices with
//      more (about 1 in 100 on meshes of fine structures, 1 in 3000 on the
//      large ones) chain the others behind and are done by k_heavy_*;
//   2. per vertex: the number of distinct neighbours and the boundary flag
//      (an edge seen in one triangle), the row lengths of each block of 256
//      rows and the slice widths summed (k_rows_count); one block scans these
//      sums (k_top_scan);
//   3. per vertex: the row (neighbours in order of first appearance, edge
//      weights accumulated in triangle order), in CSR and in its slice, the
//      lumped mass and the Gershgorin bound (k_rows_fill).
// A row is worked out in registers: its slots are sorted by a network (the
// atomics of the first pass fill them in any order), so triangles come in
// ascending order and every floating-point sum runs in a fixed order: the
// operator is the same bit for bit on every run.  For the steps the rows are
// also laid out in slices of 16 (entry e of the 16 rows of a slice side by
// side: a 64-byte line of columns, a 128-byte line of weights), so that one
// thread per row still sums its row in row order while a wave's loads of entry
// e coalesce; slices of 64 are padded to the longest of 64 rows, 32 % more
// entries on a mesh of smoothed noise against 16 % (HBM bound: the operator is read once per
// step, the field values mostly from L2 because neighbours have nearby ids).
// A mesh whose padded slices would not fit the space reserved for them steps
// on the rows.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>

#include "../../include/sbmt.h"
#include "../../include/sbmt_post.h"

namespace sbmt_pde {

constexpr int kThreads = 256;  // rows per block of the assembly, too
constexpr int kSlots = 8;      // incident triangles a vertex holds in place
constexpr int kSlice = 16;     // rows per slice of the steps' layout
constexpr int kParts = 256;    // partial extremes and counts of the rows (spread atomics)

struct Info {
  unsigned long long n_invalid;
  unsigned long long n_heavy;    // vertices of more triangles than slots
  unsigned long long heavy_used; // entries of the heavy vertices' lists
  // the result, written by k_finish
  unsigned long long min_mass_key, lambda_key;  // order keys (see order_key)
  unsigned long long n_boundary;
  long long nnz;
};
struct Part {
  unsigned long long min_mass_key, lambda_key, n_boundary;
};

__device__ __forceinline__ unsigned long long order_key(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

__device__ __forceinline__ bool tri_valid(int32_t a, int32_t b, int32_t c, int64_t nv) {
  return a >= 0 && b >= 0 && c >= 0 && a < nv && b < nv && c < nv && a != b && b != c && a != c;
}

// Half-cotangents c_k of triangle t and its cross product.
__device__ __forceinline__ double tri_weights(const double2* __restrict__ v, const int32_t* id, double c[3]) {
  double x[3], y[3];
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    const double2 p = v[id[e]];
    x[e] = p.x;
    y[e] = p.y;
  }
  const double cross = (x[1] - x[0]) * (y[2] - y[0]) - (y[1] - y[0]) * (x[2] - x[0]);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double ux = x[(k + 1) % 3] - x[k], uy = y[(k + 1) % 3] - y[k];
    const double wx = x[(k + 2) % 3] - x[k], wy = y[(k + 2) % 3] - y[k];
    c[k] = 0.5 * ((ux * wx + uy * wy) / cross);
  }
  return cross;
}

struct __attribute__((aligned(4))) Tri {
  int32_t a, b, c;
};

// ---------------------------------------------------------------------------
// Block-wide helpers.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int wave_incl_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1, 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2, 3
  return x;
}
// Largest x of the lane's slice (16 lanes).
__device__ __forceinline__ int slice_max(int x) {
#pragma unroll
  for (int off = kSlice / 2; off > 0; off >>= 1) x = max(x, __shfl_xor(x, off));
  return x;
}
// Entries of the wave's slices of the given widths (each lane its slice's).
__device__ __forceinline__ int wave_slices(int width) {
  int n = 0;
#pragma unroll
  for (int q = 0; q < 64; q += kSlice) n += __builtin_amdgcn_readlane(width, q);
  return kSlice * n;
}
__device__ __forceinline__ unsigned long long wave_min(unsigned long long x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const unsigned long long y = __shfl_xor(x, off);
    x = y < x ? y : x;
  }
  return x;
}

// Chunk of block b of a launch of xcd_blocks(n) blocks over n chunks: blocks
// go round the eight dies in turn, and each die gets one run of consecutive
// chunks, so that what neighbouring chunks share (the slots of a vertex, the
// triangles and positions around it) meets in one L2.  -1: no chunk.
constexpr unsigned kXcds = 8;
__host__ __device__ __forceinline__ unsigned xcd_blocks(int64_t n) {
  return (unsigned)((n + kXcds - 1) / kXcds) * kXcds;
}
__device__ __forceinline__ int64_t xcd_chunk(int64_t n) {
  const int64_t c = (int64_t)(blockIdx.x % kXcds) * (gridDim.x / kXcds) + blockIdx.x / kXcds;
  return c < n ? c : -1;
}

// ---------------------------------------------------------------------------
// Assembly passes.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kThreads) k_zero(int32_t* __restrict__ deg, uint32_t* __restrict__ head, int64_t n,
                                                   Part* __restrict__ part, Info* __restrict__ info) {
  const int64_t step = (int64_t)gridDim.x * kThreads;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += step) {
    deg[i] = 0;
    head[i] = 0u;
  }
  if (blockIdx.x == 0) {
    static_assert(kParts == kThreads, "one partial per thread");
    part[threadIdx.x].min_mass_key = ~0ull;
    part[threadIdx.x].lambda_key = 0ull;
    part[threadIdx.x].n_boundary = 0ull;
    if (threadIdx.x == 0) info->n_invalid = info->n_heavy = info->heavy_used = 0ull;
  }
}

// Incident triangles of every vertex: triangle t goes to slot deg[v]++ of each
// of its vertices.  256 consecutive triangles of a mesh numbered row by row
// name each of their vertices about three times, nearly all of them in two
// short ranges of ids (the two rows of the strip), and an atomic on device
// memory costs more than one on LDS: a block counts the vertices of the range
// that starts at its lowest id, and of the one that starts at the lowest id
// beyond that, in LDS and takes the places of each vertex with one atomic.
// The other vertices (a row's end, crossings numbered apart) take theirs one
// by one.  A triangle whose place lies beyond the slots is chained in front
// of the vertex's others (head: triangle + 1; next, per triangle corner, the
// head before it); the one at place kSlots lists the vertex.
constexpr int kRange = 512;
__device__ __forceinline__ int block_min(int x, int* lds) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x = min(x, __shfl_xor(x, off));
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = x;
  __syncthreads();
  return min(min(lds[0], lds[1]), min(lds[2], lds[3]));
}
__global__ void __launch_bounds__(kThreads) k_incident(const int32_t* __restrict__ tris, int64_t nt, int64_t nv,
                                                       int32_t* __restrict__ deg, int32_t* __restrict__ slots,
                                                       uint32_t* __restrict__ head, uint32_t* __restrict__ next,
                                                       int32_t* __restrict__ heavy, Info* __restrict__ info) {
  __shared__ int32_t cnt[2 * kRange];
  __shared__ int lo4[2][kThreads / 64];
  const int64_t chunk = xcd_chunk((nt + kThreads - 1) / kThreads);
  if (chunk < 0) return;  // uniform
  constexpr int kPer = 2 * kRange / kThreads;
#pragma unroll
  for (int q = 0; q < kPer; ++q) cnt[threadIdx.x + q * kThreads] = 0;
  const int64_t t = chunk * kThreads + threadIdx.x;
  Tri x = {-1, -1, -1};
  bool ok = false;
  if (t < nt) {
    x = *reinterpret_cast<const Tri*>(tris + 3 * t);
    ok = tri_valid(x.a, x.b, x.c, nv);
    if (!ok) atomicAdd(&info->n_invalid, 1ull);
  }
  constexpr int32_t kNone = 0x7fffffff;  // no vertex: ids stay below it
  const int32_t id[3] = {x.a, x.b, x.c};
  const int32_t lo0 = block_min(ok ? min(id[0], min(id[1], id[2])) : kNone, lo4[0]);
  int32_t up = kNone;
#pragma unroll
  for (int e = 0; e < 3; ++e)
    if (ok && id[e] - lo0 >= kRange) up = min(up, id[e]);
  const int32_t lo1 = block_min(up, lo4[1]);
  int at[3], place[3];
  if (ok) {
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      const int32_t r0 = id[e] - lo0, r1 = id[e] - lo1;  // lo1 <= id[e] where r0 >= kRange
      at[e] = r0 < kRange ? r0 : (r1 < kRange ? kRange + r1 : -1);
      place[e] = at[e] >= 0 ? atomicAdd(&cnt[at[e]], 1) : atomicAdd(&deg[id[e]], 1);
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int c = threadIdx.x + q * kThreads;
    const int32_t n = cnt[c];
    if (n) cnt[c] = atomicAdd(&deg[c < kRange ? lo0 + c : lo1 + (c - kRange)], n);  // the block's first place
  }
  __syncthreads();
  if (!ok) return;
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    if (at[e] >= 0) place[e] += cnt[at[e]];
    if (place[e] < kSlots) {
      slots[(int64_t)kSlots * id[e] + place[e]] = (int32_t)t;
    } else {
      next[3 * t + e] = atomicExch(&head[id[e]], (uint32_t)t + 1u);
      if (place[e] == kSlots) heavy[atomicAdd(&info->n_heavy, 1ull)] = id[e];
    }
  }
}

// The two neighbours of vertex i in triangle t (next, previous).
__device__ __forceinline__ void tri_neighbours(const int32_t* __restrict__ tris, int64_t t, int64_t i, int32_t& next,
                                               int32_t& prev) {
  const Tri x = *reinterpret_cast<const Tri*>(tris + 3 * t);
  next = x.a == i ? x.b : (x.b == i ? x.c : x.a);
  prev = x.a == i ? x.c : (x.b == i ? x.a : x.b);
}

// The slots of row i in ascending order in registers (the first deg of them;
// the rest hold INT32_MAX), by a sorting network of 19 exchanges.
__device__ __forceinline__ void load_slots(const int32_t* __restrict__ slots, int64_t i, int deg, int32_t (&t)[kSlots]) {
  const int4* p = reinterpret_cast<const int4*>(slots + kSlots * i);
  const int4 a = p[0], b = p[1];
  const int32_t raw[kSlots] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
  for (int e = 0; e < kSlots; ++e) t[e] = e < deg ? raw[e] : 0x7fffffff;
  constexpr int8_t net[19][2] = {{0, 2}, {1, 3}, {4, 6}, {5, 7}, {0, 4}, {1, 5}, {2, 6}, {3, 7}, {0, 1}, {2, 3},
                                 {4, 5}, {6, 7}, {2, 4}, {3, 5}, {1, 4}, {3, 6}, {1, 2}, {3, 4}, {5, 6}};
#pragma unroll
  for (int q = 0; q < 19; ++q) {
    const int32_t lo = min(t[net[q][0]], t[net[q][1]]), hi = max(t[net[q][0]], t[net[q][1]]);
    t[net[q][0]] = lo;
    t[net[q][1]] = hi;
  }
}

// The 2 deg neighbour candidates of row i in order (triangles ascending, next
// then previous); places beyond them hold values that occur nowhere else.
// Every triangle is loaded before the first is looked at (one wait for all of
// them; places beyond deg load one that is there).
__device__ __forceinline__ void load_candidates(const int32_t* __restrict__ tris, int64_t i, int deg,
                                                const int32_t (&t)[kSlots], int32_t (&j)[2 * kSlots],
                                                bool (&k0)[kSlots], bool (&k1)[kSlots]) {
  Tri x[kSlots];
#pragma unroll
  for (int e = 0; e < kSlots; ++e)
    x[e] = *reinterpret_cast<const Tri*>(tris + 3 * (int64_t)(e < deg ? t[e] : (deg > 0 ? t[0] : 0)));
#pragma unroll
  for (int e = 0; e < kSlots; ++e) {
    k0[e] = x[e].a == i;
    k1[e] = x[e].b == i;
    const int32_t n = k0[e] ? x[e].b : (k1[e] ? x[e].c : x[e].a), p = k0[e] ? x[e].c : (k1[e] ? x[e].a : x[e].b);
    j[2 * e] = e < deg ? n : -2 - 2 * e;
    j[2 * e + 1] = e < deg ? p : -3 - 2 * e;
  }
}

// Distinct neighbours of a row and whether one of them occurs once.
__device__ __forceinline__ void count_row(const int32_t* __restrict__ tris, int64_t i, int deg,
                                          const int32_t (&t)[kSlots], int& uniq, bool& boundary) {
  int32_t j[2 * kSlots];
  bool k0[kSlots], k1[kSlots];
  load_candidates(tris, i, deg, t, j, k0, k1);
  uint32_t dup = 0, mate = 0;  // candidates with an equal one before them; with any equal one
#pragma unroll
  for (int p = 1; p < 2 * kSlots; ++p)
#pragma unroll
    for (int q = 0; q < p; ++q) {
      const bool eq = j[p] == j[q];
      dup |= eq ? 1u << p : 0u;
      mate |= eq ? (1u << p) | (1u << q) : 0u;
    }
  uniq = 2 * deg - __builtin_popcount(dup);
  boundary = mate != (1u << (2 * deg)) - 1u;
}

// The heavy vertices, a wave each: 64 of a row's candidates (candidate p: the next
// or the previous neighbour in triangle p / 2 of the sorted list) lie in the wave's
// lanes at a time, and the others pass by 64 at a time, lane by lane.  This one
// collects and sorts the lists, counts the rows and flags the boundary.  The list's
// place takes the slots' (they are copied).
// The work is quadratic in a row's triangles, so what bounds it is how many lanes
// share it: assembling 100000 vertices of 40 triangles of random vertices took 14.7 ms
// with a lane per vertex, 177 with everything beyond 32 triangles left to lane 0, now
// 4.1; 20000 vertices of 100 triangles 45, 858, now 12; 50000 closed fans of 40
// triangles 21.9, 31.8, now 1.8.
__device__ __forceinline__ int32_t candidate(const int32_t* __restrict__ tris, const int32_t* list, int32_t i, int32_t d,
                                             int32_t p) {
  int32_t n = -1, q = -1;
  if (p < 2 * (int64_t)d) tri_neighbours(tris, list[p >> 1], i, n, q);
  return (p & 1) ? q : n;
}
__global__ void __launch_bounds__(kThreads) k_heavy_count(const int32_t* __restrict__ tris,
                                                          const int32_t* __restrict__ deg,
                                                          int32_t* __restrict__ slots,
                                                          const uint32_t* __restrict__ head,
                                                          const uint32_t* __restrict__ next,
                                                          const int32_t* __restrict__ heavy, int32_t* inc,
                                                          int32_t* scratch, int32_t* __restrict__ row_len,
                                                          uint8_t* __restrict__ bnd, Info* __restrict__ info) {
  const int64_t n = (int64_t)info->n_heavy, step = (int64_t)gridDim.x * (kThreads / 64);
  const int lane = threadIdx.x & 63;
  for (int64_t h = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6); h < n; h += step) {
    const int32_t i = heavy[h], d = deg[i];
    unsigned long long at = 0;
    if (lane == 0) at = atomicAdd(&info->heavy_used, (unsigned long long)d);
    at = __shfl(at, 0);
    int32_t* const list = inc + at;
    // the chained triangles after the slots' (a link's corners and the heads before
    // it are asked for together: one wait a link)
    int32_t m = kSlots;
    for (uint32_t c = head[i]; c && m < d; ++m) {
      const int64_t t = (int64_t)c - 1;
      const Tri x = *reinterpret_cast<const Tri*>(tris + 3 * t);
      const uint32_t c0 = next[3 * t], c1 = next[3 * t + 1], c2 = next[3 * t + 2];
      if (lane == 0) list[m] = (int32_t)t;
      c = x.a == i ? c0 : (x.b == i ? c1 : c2);
    }
    if (lane < kSlots) list[lane] = slots[(int64_t)kSlots * i + lane];
    __threadfence_block();
    // sorted: triangles are distinct, a place is the number of smaller ones (up to
    // 64 are all read before the first is put in place, more go through `scratch`,
    // the same range of it as of `inc`)
    int32_t* const to = d <= 64 ? list : scratch + at;
    for (int32_t p0 = 0; p0 < d; p0 += 64) {
      const bool is = lane < d - p0;
      const int32_t t = is ? list[p0 + lane] : 0x7fffffff;
      int32_t place = 0;
      for (int32_t q0 = 0; q0 < d; q0 += 64) {
        const int32_t x = q0 == p0 ? t : (lane < d - q0 ? list[q0 + lane] : 0x7fffffff);
        for (int q = 0; q < min(64, d - q0); ++q) place += __builtin_amdgcn_readlane(x, q) < t;
      }
      if (is) to[place] = t;
    }
    __threadfence_block();
    if (to != list) {
      for (int32_t p = lane; p < d; p += 64) list[p] = to[p];
      __threadfence_block();
    }
    int32_t uniq = 0;
    bool boundary = false;
    for (int32_t p0 = 0; p0 < 2 * d; p0 += 64) {
      const bool is = lane < 2 * d - p0;
      const int32_t j = candidate(tris, list, i, d, p0 + lane);
      int mult = 0;
      bool first = is;
      for (int32_t q0 = 0; q0 < 2 * d; q0 += 64) {
        const int32_t x = q0 == p0 ? j : candidate(tris, list, i, d, q0 + lane);
        for (int q = 0; q < min(64, 2 * d - q0); ++q) {
          const bool eq = __builtin_amdgcn_readlane(x, q) == j;
          mult += eq;
          first = first && !(eq && q0 + q < p0 + lane);
        }
      }
      uniq += (int32_t)__popcll(__ballot(first));
      boundary = boundary || __ballot(is && mult == 1) != 0ull;
    }
    if (lane == 0) {
      row_len[i] = uniq;
      bnd[i] = boundary ? 1 : 0;
      *reinterpret_cast<int64_t*>(slots + (int64_t)kSlots * i) = (int64_t)at;
    }
  }
}

// Row lengths and boundary flags; per block the entries of its 256 rows and of
// its slices (16 times the longest row of each).
__global__ void __launch_bounds__(kThreads) k_rows_count(const int32_t* __restrict__ tris, int64_t nv,
                                                         const int32_t* __restrict__ deg,
                                                         const int32_t* __restrict__ slots,
                                                         int32_t* __restrict__ row_len, uint8_t* __restrict__ bnd,
                                                         longlong2* __restrict__ bsum, Part* __restrict__ part) {
  __shared__ int len4[kThreads / 64], wid4[kThreads / 64], bnd4[kThreads / 64];
  const int64_t blk = xcd_chunk((nv + kThreads - 1) / kThreads);
  if (blk < 0) return;  // uniform
  const int64_t i = blk * kThreads + threadIdx.x;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int d = i < nv ? deg[i] : 0;
  int len = 0;
  bool boundary = false;
  if (d > kSlots) {
    len = row_len[i];
    boundary = bnd[i] != 0;
  }
  const int dl = d <= kSlots ? d : 0;
  int32_t t[kSlots];
  load_slots(slots, i < nv ? i : 0, dl, t);
  if (__ballot(dl > 0) != 0ull) {  // uniform: there is a triangle to load
    int lc = 0;
    bool bc = false;
    count_row(tris, i, dl, t, lc, bc);
    if (dl > 0) {
      len = lc;
      boundary = bc;
    }
  }
  if (i < nv && d <= kSlots) {
    row_len[i] = len;
    bnd[i] = boundary ? 1 : 0;
  }
  const int tot = __builtin_amdgcn_readlane(wave_incl_scan(len), 63), wid = wave_slices(slice_max(len));
  const int nb = (int)__popcll(__ballot(boundary));
  if (lane == 0) {
    len4[wv] = tot;
    wid4[wv] = wid;
    bnd4[wv] = nb;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    long long a = 0, b = 0;
    int c = 0;
    for (int w = 0; w < kThreads / 64; ++w) {
      a += len4[w];
      b += wid4[w];
      c += bnd4[w];
    }
    bsum[blk] = make_longlong2(a, b);
    if (c) atomicAdd(&part[blk & (kParts - 1)].n_boundary, (unsigned long long)c);
  }
}

// One workgroup: exclusive scan of the blocks' sums in place; the totals go
// behind the last one and to the ends of both offset arrays.
constexpr int kTop = 1024, kTopPer = 8;
__global__ void __launch_bounds__(kTop) k_top_scan(longlong2* __restrict__ bsum, int64_t nb,
                                                   int64_t* __restrict__ row_end, int64_t* __restrict__ slice_end) {
  __shared__ long long sa[kTop / 64], sb[kTop / 64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  long long ra = 0, rb = 0;  // the sums before this round's blocks
  for (int64_t base = 0; base < nb; base += kTopPer * kTop) {
    const int64_t lo = base + kTopPer * (int64_t)threadIdx.x;
    longlong2 v[kTopPer];
    long long a = 0, b = 0;
#pragma unroll
    for (int q = 0; q < kTopPer; ++q) {
      v[q] = lo + q < nb ? bsum[lo + q] : make_longlong2(0, 0);
      a += v[q].x;
      b += v[q].y;
    }
    long long ia = a, ib = b;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const long long ya = __shfl_up(ia, off), yb = __shfl_up(ib, off);
      if (lane >= off) {
        ia += ya;
        ib += yb;
      }
    }
    if (lane == 63) {
      sa[wv] = ia;
      sb[wv] = ib;
    }
    __syncthreads();
    long long ea = ra + ia - a, eb = rb + ib - b;
    for (int w = 0; w < kTop / 64; ++w) {
      ea += w < wv ? sa[w] : 0;
      eb += w < wv ? sb[w] : 0;
      ra += sa[w];
      rb += sb[w];
    }
#pragma unroll
    for (int q = 0; q < kTopPer; ++q) {
      if (lo + q < nb) bsum[lo + q] = make_longlong2(ea, eb);
      ea += v[q].x;
      eb += v[q].y;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *row_end = ra;
    *slice_end = rb;
  }
}

// Where a heavy vertex's row goes: CSR from r0, and entry e of its slice at s0 + 16 e.
struct RowOut {
  int32_t* col;
  double* val;
  int32_t* col_s;  // nullptr when the slices do not fit
  double* val_s;
  int64_t r0, s0;
};
__device__ __forceinline__ void put_entry(const RowOut& o, int e, int32_t j, double w) {
  o.col[o.r0 + e] = j;
  o.val[o.r0 + e] = w;
  if (o.col_s) {
    o.col_s[o.s0 + kSlice * (int64_t)e] = j;
    o.val_s[o.s0 + kSlice * (int64_t)e] = w;
  }
}

// Rows a wave works out in LDS at a time: the entries of 64 rows of eight.
constexpr int kStage = 512;

// Row i from its sorted triangles into its place in the staged entries (col,
// val): candidate by candidate, a neighbour seen before adds its weight to its
// entry, a new one takes the next.  Returns the mass.
__device__ __forceinline__ double make_row(const double2* __restrict__ v, const int32_t* __restrict__ tris, int64_t i,
                                           int deg, const int32_t (&t)[kSlots], int32_t* col, double* val) {
  int32_t j[2 * kSlots];
  bool k0[kSlots], k1[kSlots];
  load_candidates(tris, i, deg, t, j, k0, k1);
  const double2 c = v[i];
  double m = 0.0;
  uint64_t place = 0;  // nibble p: the entry of candidate p
  uint32_t n = 0;      // entries so far
  constexpr int kAtOnce = 2;  // triangles whose positions are loaded together (four: more registers, fewer waves)
#pragma unroll
  for (int h = 0; h < kSlots; h += kAtOnce) {
    double2 pos[2 * kAtOnce];
#pragma unroll
    for (int a = 0; a < 2 * kAtOnce; ++a) pos[a] = v[2 * h + a < 2 * deg ? j[2 * h + a] : (int32_t)i];
#pragma unroll
    for (int e = h; e < h + kAtOnce; ++e) {
      if (e >= deg) continue;
      // triangle by triangle as tri_weights computes it: the cross product in
      // the triangle's own vertex order, the half-cotangents opposite i's two edges
      const double2 q = pos[2 * (e - h)], p = pos[2 * (e - h) + 1];  // next, previous
      const double cpx = c.x - p.x, cpy = c.y - p.y, qpx = q.x - p.x, qpy = q.y - p.y;
      const double cqx = c.x - q.x, cqy = c.y - q.y, pqx = p.x - q.x, pqy = p.y - q.y;
      // i in place 0: (q - c) x (p - c) = (c - q) x (c - p); in place 1:
      // (c - p) x (q - p); in place 2: (p - q) x (c - q) = (c - q) x (q - p),
      // the same products and so the same roundings
      const double ux = k1[e] ? cpx : cqx, uy = k1[e] ? cpy : cqy, wx = k0[e] ? cpx : qpx, wy = k0[e] ? cpy : qpy;
      double cross = ux * wy - uy * wx;
      if (cross == 0.0) {  // a triangle without area: the sign of the zero decides those of its infinite weights
        const double2 x0 = k0[e] ? c : (k1[e] ? p : q), x1 = k0[e] ? q : (k1[e] ? c : p), x2 = k0[e] ? p : (k1[e] ? q : c);
        cross = (x1.x - x0.x) * (x2.y - x0.y) - (x1.y - x0.y) * (x2.x - x0.x);
      }
      const double w[2] = {0.5 * ((cpx * qpx + cpy * qpy) / cross),   // angle at the previous vertex
                           0.5 * ((pqx * cqx + pqy * cqy) / cross)};  // at the next one
      m += (0.5 * cross) / 3.0;
#pragma unroll
      for (int z = 0; z < 2; ++z) {
        const int b = 2 * e + z;
        int first = b;
#pragma unroll
        for (int a = b - 1; a >= 0; --a) first = j[a] == j[b] ? a : first;
        const bool fresh = first == b;
        const uint32_t at = fresh ? n : (uint32_t)(place >> (4 * first)) & 15u;
        place |= (uint64_t)at << (4 * b);
        n += fresh ? 1u : 0u;
        const double before = val[at];
        val[at] = fresh ? w[z] : before + w[z];
        if (fresh) col[at] = j[b];
      }
    }
  }
  return m;
}

__device__ __forceinline__ unsigned long long lambda_of(double diag, double offs, double m) {
  if (!(m > 0.0)) return 0ull;
  const double lam = (diag + offs) / m;
  return isnan(lam) ? 0ull : order_key(lam);
}

// Offsets, rows and masses, a wave (and a block) per 64 rows.  The
// time goes into a chain of loads (slots, triangles, positions) that only
// other waves hide, so blocks of one wave (a block of four holds its LDS
// until the last is done: 745 us on 8.4 M rows) and at most 128 registers
// (152 without the bound: 600 us against 530 for the same rows).  The CSR
// entries of the 64 rows are one run, written as such from LDS (a row per
// lane would touch every line of the run once per entry), unless a heavy row
// lies between them.  The padding of a slice (rows shorter than its longest)
// points at the row itself with weight 0: the steps load it without a test
// and leave it out of the sum.
__global__ void __launch_bounds__(64, 4) k_rows_fill(
    const double2* __restrict__ v, const int32_t* __restrict__ tris, int64_t nv, const int32_t* __restrict__ deg,
    const int32_t* __restrict__ slots, const int32_t* __restrict__ row_len, const longlong2* __restrict__ bsum,
    int64_t nsl, int64_t cap, int64_t* __restrict__ row_off, int64_t* __restrict__ slice_off, int32_t* __restrict__ col,
    double* __restrict__ val, int32_t* __restrict__ col_s, double* __restrict__ val_s, double* __restrict__ mass,
    Part* __restrict__ part) {
  __shared__ int32_t st_col[kStage];
  __shared__ double st_val[kStage];
  const int64_t group = xcd_chunk((nv + 63) / 64);
  if (group < 0) return;  // uniform
  const int lane = threadIdx.x;
  const int64_t i = 64 * group + lane;
  const int d = i < nv ? deg[i] : 0;
  const bool light = i < nv && d <= kSlots;
  const int dl = light ? d : 0;
  // the block of 256 rows these 64 are part of: the rows before them
  constexpr int kPer = kThreads / 64;
  const int before = (int)(group % kPer);
  const longlong2 b = bsum[group / kPer];
  const bool sliced = slice_off[nsl] <= cap;  // uniform
  const int len = i < nv ? row_len[i] : 0;
  int lens[kPer - 1];
#pragma unroll
  for (int w = 0; w < kPer - 1; ++w) lens[w] = w < before ? row_len[i - 64 * (before - w)] : 0;
  int64_t r0 = b.x, s0 = b.y;  // the first entry of the 64 rows, of their slices
#pragma unroll
  for (int w = 0; w < kPer - 1; ++w)
    if (w < before) {
      r0 += __builtin_amdgcn_readlane(wave_incl_scan(lens[w]), 63);
      s0 += wave_slices(slice_max(lens[w]));
    }
  const int incl = wave_incl_scan(len), wid = slice_max(len);
  for (int q = 0; q < 64 / kSlice - 1; ++q)  // this lane's place in its slice
    s0 += q < lane / kSlice ? kSlice * __builtin_amdgcn_readlane(wid, kSlice * q) : 0;
  s0 += lane % kSlice;
  const int64_t row = r0 + (incl - len);
  if (i < nv) row_off[i] = row;
  if (lane % kSlice == 0 && i < nv) slice_off[i / kSlice] = s0;
  const int ll = light ? len : 0;
  const int lincl = wave_incl_scan(ll), lat = lincl - ll;  // places among the light rows
  const int ltotal = __builtin_amdgcn_readlane(lincl, 63);
  const bool one_run = __ballot(i < nv && !light) == 0ull;
  int32_t t[kSlots];
  load_slots(slots, i < nv ? i : 0, dl, t);
  double m = 0.0, diag = 0.0, offs = 0.0;
  // once, or over the rows that fit from place `start` on (a row has at most
  // 16 entries, so every round takes some)
  for (int start = 0; start == 0 || start < ltotal;) {  // uniform
    const bool in = ll > 0 && lat >= start && lat + ll <= start + kStage;
    int32_t* const sc = &st_col[lat - start];
    double* const sv = &st_val[lat - start];
    if (in) m = make_row(v, tris, i, dl, t, sc, sv);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // the slice's entries with their padding (whole lines but for the rows of
    // another round), the sums of the row
    const bool put = sliced && (in || (ll == 0 && start == 0));
    for (int e = 0; e < wid; ++e) {  // the same in the lanes of a slice
      const bool has = in && e < ll;
      const double x = has ? sv[e] : 0.0;
      const int32_t j = has ? sc[e] : (int32_t)i;
      diag = has ? diag + x : diag;
      offs = has ? offs + fabs(x) : offs;
      if (put) {
        col_s[s0 + kSlice * (int64_t)e] = j;
        val_s[s0 + kSlice * (int64_t)e] = x;
      }
      if (!one_run && has) {
        col[row + e] = j;
        val[row + e] = x;
      }
    }
    const unsigned long long rest = __ballot(ll > 0 && lat + ll > start + kStage);
    const int next = rest ? __builtin_amdgcn_readlane(lat, __builtin_ctzll(rest)) : max(ltotal, 1);
    if (one_run)
      for (int x = lane; x < min(next, ltotal) - start; x += 64) {
        col[r0 + start + x] = st_col[x];
        val[r0 + start + x] = st_val[x];
      }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    start = next;
  }
  unsigned long long mn = ~0ull, mx = 0ull;
  if (light) {
    mass[i] = m;
    if (!isnan(m)) mn = order_key(m);
    mx = lambda_of(diag, offs, m);
  }
  mn = wave_min(mn);
  mx = ~wave_min(~mx);
  if (lane == 0) {
    Part* const q = &part[group & (kParts - 1)];
    atomicMin(&q->min_mass_key, mn);
    atomicMax(&q->lambda_key, mx);
  }
}

// Candidate p of heavy vertex i: its weight, its neighbour j and its triangle's share
// of the mass.
__device__ __forceinline__ double candidate_weight(const double2* __restrict__ v, const int32_t* __restrict__ tris,
                                                   const int32_t* __restrict__ list, int32_t i, int32_t d, int32_t p,
                                                   int32_t& j, double& share) {
  j = -1;
  share = 0.0;
  if (p >= 2 * (int64_t)d) return 0.0;
  const Tri x = *reinterpret_cast<const Tri*>(tris + 3 * (int64_t)list[p >> 1]);
  const int32_t id[3] = {x.a, x.b, x.c};
  double c[3];
  share = (0.5 * tri_weights(v, id, c)) / 3.0;
  const int k = x.a == i ? 0 : (x.b == i ? 1 : 2), z = (p & 1) ? (k + 1) % 3 : (k + 2) % 3;  // opposite the edge
  j = (p & 1) ? (k == 0 ? x.c : (k == 1 ? x.a : x.b)) : (k == 0 ? x.b : (k == 1 ? x.c : x.a));
  return z == 0 ? c[0] : (z == 1 ? c[1] : c[2]);
}
// x of lane q (uniform).
__device__ __forceinline__ double lane_value(double x, int q) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, q);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), q);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// The heavy vertices' rows, from their sorted lists, a wave each.
__global__ void __launch_bounds__(kThreads) k_heavy_fill(const double2* __restrict__ v, const int32_t* __restrict__ tris,
                                                         const int32_t* __restrict__ deg,
                                                         const int32_t* __restrict__ slots,
                                                         const int32_t* __restrict__ heavy,
                                                         const int32_t* __restrict__ inc,
                                                         const int64_t* __restrict__ row_off,
                                                         const int64_t* __restrict__ slice_off, int64_t nsl, int64_t cap,
                                                         int32_t* __restrict__ col, double* __restrict__ val,
                                                         int32_t* __restrict__ col_s, double* __restrict__ val_s,
                                                         double* __restrict__ mass, Part* __restrict__ part,
                                                         const Info* __restrict__ info) {
  const int64_t n = (int64_t)info->n_heavy, step = (int64_t)gridDim.x * (kThreads / 64);
  const bool sliced = slice_off[nsl] <= cap;  // uniform
  const int lane = threadIdx.x & 63;
  for (int64_t h = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6); h < n; h += step) {
    const int32_t i = heavy[h], d = deg[i];
    const int32_t* const list = inc + *reinterpret_cast<const int64_t*>(slots + (int64_t)kSlots * i);
    RowOut o;
    o.col = col;
    o.val = val;
    o.col_s = sliced ? col_s : nullptr;
    o.val_s = val_s;
    o.r0 = row_off[i];
    o.s0 = slice_off[i / kSlice] + i % kSlice;
    double m = 0.0, diag = 0.0, offs = 0.0;
    int e0 = 0;  // entries so far
    for (int32_t p0 = 0; p0 < 2 * d; p0 += 64) {
      // lane l: neighbour and weight of candidate p0 + l, and its triangle's share of the mass
      int32_t j;
      double share;
      double w = candidate_weight(v, tris, list, i, d, p0 + lane, j, share);
      const double own = w;
      bool first = lane < 2 * d - p0;
      for (int32_t q0 = 0; q0 < 2 * d; q0 += 64) {
        int32_t x = j;
        double wx = own, sx;
        if (q0 != p0) wx = candidate_weight(v, tris, list, i, d, q0 + lane, x, sx);
        for (int q = 0; q < min(64, 2 * d - q0); ++q) {
          const double wq = lane_value(wx, q);
          if (__builtin_amdgcn_readlane(x, q) == j) {
            w = q0 + q > p0 + lane ? w + wq : w;
            first = first && q0 + q >= p0 + lane;
          }
        }
      }
      for (int e = 0; e < min(64, 2 * d - p0); e += 2) m += lane_value(share, e);
      const unsigned long long rows = __ballot(first);
      const int e = e0 + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(rows >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)rows, 0u));
      if (first) put_entry(o, e, j, w);
      e0 += (int)__popcll(rows);
      for (unsigned long long r = rows; r; r &= r - 1) {
        const double x = lane_value(w, __builtin_ctzll(r));
        diag += x;
        offs += fabs(x);
      }
    }
    if (lane == 0) {
      mass[i] = m;
      Part* const q = &part[h & (kParts - 1)];
      if (!isnan(m)) atomicMin(&q->min_mass_key, order_key(m));
      atomicMax(&q->lambda_key, lambda_of(diag, offs, m));
    }
  }
}

// The summary from the partial results.
__global__ void __launch_bounds__(kParts) k_finish(const Part* __restrict__ part, const int64_t* __restrict__ row_end,
                                                   Info* __restrict__ info) {
  __shared__ unsigned long long mn4[kParts / 64], mx4[kParts / 64], nb4[kParts / 64];
  const Part p = part[threadIdx.x];
  const unsigned long long mn = wave_min(p.min_mass_key), mx = wave_min(~p.lambda_key);
  unsigned long long nb = p.n_boundary;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) nb += __shfl_xor(nb, off);
  if ((threadIdx.x & 63) == 0) {
    mn4[threadIdx.x >> 6] = mn;
    mx4[threadIdx.x >> 6] = mx;
    nb4[threadIdx.x >> 6] = nb;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  unsigned long long a = ~0ull, b = ~0ull, c = 0ull;
  for (int w = 0; w < kParts / 64; ++w) {
    a = mn4[w] < a ? mn4[w] : a;
    b = mx4[w] < b ? mx4[w] : b;
    c += nb4[w];
  }
  info->min_mass_key = a;
  info->lambda_key = ~b;
  info->n_boundary = c;
  info->nnz = *row_end;
}

// ---------------------------------------------------------------------------
// Operator application and heat steps.
// ---------------------------------------------------------------------------
struct Op {  // what an application of the operator reads
  const int64_t* row_off;
  const int32_t* col;
  const double* val;
  const int32_t* row_len;
  const int64_t* slice_off;
  const int32_t* col_s;
  const double* val_s;
  const double* mass;
  const uint8_t* bnd;
  int64_t nsl, cap;
};

// (K u)_i in row order from the CSR rows.
__device__ __forceinline__ double csr_row(const Op& op, int64_t i, double ui, const double* __restrict__ u) {
  double s = 0.0;
  for (int64_t e = op.row_off[i], end = op.row_off[i + 1]; e < end; ++e) s += op.val[e] * (ui - u[op.col[e]]);
  return s;
}
// (K u)_i of a heat step, the same sum; 0 of a row that is held, whose entries are
// not loaded (on a mesh of fine structures two rows in three: 2.0 M vertices 67 us
// with them, 56 without; one in ten, 2.7 M vertices: 51 either way).  In slices the
// entries of a row are loaded kAhead at a time, columns, weights, then the field
// values, so that a wave waits for memory once per kAhead entries and not once per
// entry; the slice's padding is loaded with them (the same line for all its rows)
// and not summed.
constexpr int kAhead = 4;
__device__ __forceinline__ double step_row(const Op& op, bool sliced, bool held, int64_t i, double ui,
                                           const double* __restrict__ u) {
  double s = 0.0;
  if (sliced) {
    const int64_t q = i / kSlice, s0 = op.slice_off[q];
    const int width = (int)(op.slice_off[q + 1] - s0) / kSlice, len = op.row_len[i], end = held ? 0 : width;
    const int32_t* const c = op.col_s + s0 + i % kSlice;
    const double* const w = op.val_s + s0 + i % kSlice;
    for (int e = 0; e < end; e += kAhead) {
      int32_t cj[kAhead];
      double wj[kAhead], uj[kAhead];
#pragma unroll
      for (int a = 0; a < kAhead; ++a) {
        const int x = min(e + a, width - 1);
        cj[a] = c[kSlice * x];
        wj[a] = w[kSlice * x];
      }
#pragma unroll
      for (int a = 0; a < kAhead; ++a) uj[a] = u[cj[a]];
#pragma unroll
      for (int a = 0; a < kAhead; ++a) s = e + a < len ? s + wj[a] * (ui - uj[a]) : s;
    }
  } else if (!held) {
    s = csr_row(op, i, ui, u);
  }
  return s;
}

// Reads the CSR arrays and not the steps' copy of them: sbmt_laplacian_csr hands
// those out, and what a program writes to them is what it applies.
__global__ void __launch_bounds__(kThreads) k_apply(Op op, int64_t nv, const double* __restrict__ u,
                                                    double* __restrict__ y) {
  const int64_t step = (int64_t)gridDim.x * kThreads;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < nv; i += step)
    y[i] = csr_row(op, i, u[i], u);
}

__global__ void __launch_bounds__(kThreads) k_heat_step(Op op, int64_t nv, double dt_alpha,
                                                        const double* __restrict__ u, double* __restrict__ out) {
  const bool sliced = op.slice_off[op.nsl] <= op.cap;  // uniform
  const int64_t step = (int64_t)gridDim.x * kThreads;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < nv; i += step) {
    const double ui = u[i], m = op.mass[i];
    const bool held = op.bnd[i] != 0;
    const double s = step_row(op, sliced, held, i, ui, u);
    out[i] = held ? 0.0 : ui - (dt_alpha * s) / m;
  }
}

__global__ void __launch_bounds__(kThreads) k_heat_init(const double2* __restrict__ v, const uint8_t* __restrict__ bnd,
                                                        int64_t nv, double x0, double y0, double sigma, double amp,
                                                        double* __restrict__ u) {
  const int64_t step = (int64_t)gridDim.x * kThreads;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < nv; i += step) {
    const double2 p = v[i];
    const double dx = p.x - x0, dy = p.y - y0;
    u[i] = bnd[i] ? 0.0 : amp * exp(-(dx * dx + dy * dy) / (2.0 * sigma * sigma));
  }
}

__global__ void __launch_bounds__(kThreads) k_copy(const double* __restrict__ a, int64_t n, double* __restrict__ b) {
  const int64_t step = (int64_t)gridDim.x * kThreads;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += step) b[i] = a[i];
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct Layout {
  size_t info, part, deg, head, heavy, slots, inc, row_len, row_off, col, val, mass, bnd, bsum, slice_off, col_s, val_s, total;
  int64_t nsl, nblk, cap;
};

static Layout layout(int64_t nv, int64_t nt) {
  Layout L;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o += align256(bytes);
    return at;
  };
  L.nsl = (nv + kSlice - 1) / kSlice;
  L.nblk = (nv + kThreads - 1) / kThreads;
  L.info = take(sizeof(Info));
  L.part = take(kParts * sizeof(Part));
  L.deg = take(4 * (size_t)nv);
  L.head = take(4 * (size_t)nv);
  L.heavy = take(4 * (size_t)std::min(nv, nt / 3 + 1));  // nine triangles or more each
  L.slots = take(4 * kSlots * (size_t)nv);
  L.inc = take(4 * 3 * (size_t)nt);  // the heavy vertices' lists
  L.row_len = take(4 * (size_t)nv);
  L.row_off = take(8 * (size_t)(nv + 1));
  L.col = take(4 * 6 * (size_t)nt);  // at most two distinct neighbours per incident triangle
  L.val = take(8 * 6 * (size_t)nt);
  L.mass = take(8 * (size_t)nv);
  L.bnd = take((size_t)nv);
  L.bsum = take(16 * (size_t)(L.nblk + 1));
  L.cap = 6 * nt;  // as many entries as the rows may hold: padding beyond twice the entries falls back
  L.slice_off = take(8 * (size_t)(L.nsl + 1));
  L.col_s = take(4 * (size_t)L.cap);
  L.val_s = take(8 * (size_t)L.cap);  // until the rows are filled: a word per triangle corner (chained triangles)
  L.total = o;
  return L;
}

static int grid_for(int64_t n) {
  const int64_t b = (n + kThreads - 1) / kThreads;
  return (int)(b < 1 ? 1 : (b > 65536 ? 65536 : b));
}

static Op op_of(const char* w, const Layout& L) {
  Op op;
  op.row_off = (const int64_t*)(w + L.row_off);
  op.col = (const int32_t*)(w + L.col);
  op.val = (const double*)(w + L.val);
  op.row_len = (const int32_t*)(w + L.row_len);
  op.slice_off = (const int64_t*)(w + L.slice_off);
  op.col_s = (const int32_t*)(w + L.col_s);
  op.val_s = (const double*)(w + L.val_s);
  op.mass = (const double*)(w + L.mass);
  op.bnd = (const uint8_t*)(w + L.bnd);
  op.nsl = L.nsl;
  op.cap = L.cap;
  return op;
}

static double host_key_value(unsigned long long k) {
  const unsigned long long b = (k >> 63) ? (k & 0x7fffffffffffffffull) : ~k;
  double d;
  memcpy(&d, &b, sizeof d);
  return d;
}

static bool sizes_ok(int64_t nv, int64_t nt) { return nv >= 0 && nt >= 0 && nv <= 0x7fffffffLL && nt <= 0x7fffffffLL; }

}  // namespace sbmt_pde

using namespace sbmt_pde;

extern "C" {

sbmt_status sbmt_laplacian_workspace(int64_t n_vertices, int64_t n_triangles, size_t* bytes) {
  if (!bytes || !sizes_ok(n_vertices, n_triangles)) return SBMT_E_INVALID_ARG;
  *bytes = layout(n_vertices, n_triangles).total;
  return SBMT_OK;
}

sbmt_status sbmt_laplacian_csr(void* workspace, size_t ws_bytes, int64_t n_vertices, int64_t n_triangles,
                               sbmt_csr* out) {
  if (!out || !sizes_ok(n_vertices, n_triangles)) return SBMT_E_INVALID_ARG;
  const Layout L = layout(n_vertices, n_triangles);
  if (!workspace || ws_bytes < L.total) return SBMT_E_WORKSPACE;
  char* w = (char*)workspace;
  out->row_off = (const int64_t*)(w + L.row_off);
  out->col = (const int32_t*)(w + L.col);
  out->val = (const double*)(w + L.val);
  out->mass = (const double*)(w + L.mass);
  out->boundary = (const uint8_t*)(w + L.bnd);
  return SBMT_OK;
}

sbmt_status sbmt_laplacian_assemble(sbmt_handle h, const double* verts, int64_t n_vertices, const int32_t* tris,
                                    int64_t n_triangles, void* workspace, size_t ws_bytes,
                                    sbmt_laplacian_info* info, void* stream) {
  if (!h || !info || !sizes_ok(n_vertices, n_triangles)) return SBMT_E_INVALID_ARG;
  if ((n_vertices > 0 && !verts) || (n_triangles > 0 && !tris)) return SBMT_E_INVALID_ARG;
  const Layout L = layout(n_vertices, n_triangles);
  if (!workspace || ws_bytes < L.total) return SBMT_E_WORKSPACE;
  char* w = (char*)workspace;
  hipStream_t s = (hipStream_t)stream;
  Info* dinfo = (Info*)(w + L.info);
  Part* part = (Part*)(w + L.part);
  int32_t* deg = (int32_t*)(w + L.deg);
  uint32_t* head = (uint32_t*)(w + L.head);
  int32_t* heavy = (int32_t*)(w + L.heavy);
  int32_t* slots = (int32_t*)(w + L.slots);
  int32_t* inc = (int32_t*)(w + L.inc);
  int32_t* row_len = (int32_t*)(w + L.row_len);
  int64_t* row_off = (int64_t*)(w + L.row_off);
  int32_t* col = (int32_t*)(w + L.col);
  double* val = (double*)(w + L.val);
  double* mass = (double*)(w + L.mass);
  uint8_t* bnd = (uint8_t*)(w + L.bnd);
  longlong2* bsum = (longlong2*)(w + L.bsum);
  int64_t* slice_off = (int64_t*)(w + L.slice_off);
  int32_t* col_s = (int32_t*)(w + L.col_s);
  double* val_s = (double*)(w + L.val_s);
  const double2* v = (const double2*)verts;
  uint32_t* next = (uint32_t*)val_s;  // scratch in the slices' room, which is written last
  hipLaunchKernelGGL(k_zero, dim3(grid_for(n_vertices)), dim3(kThreads), 0, s, deg, head, n_vertices, part, dinfo);
  const dim3 hgrid((unsigned)std::min<int64_t>(std::max<int64_t>(L.nblk, 1), 2048));  // heavy vertices are few
  if (n_triangles > 0) {
    hipLaunchKernelGGL(k_incident, dim3(xcd_blocks((n_triangles + kThreads - 1) / kThreads)), dim3(kThreads), 0, s, tris, n_triangles, n_vertices,
                       deg, slots, head, next, heavy, dinfo);
    hipLaunchKernelGGL(k_heavy_count, hgrid, dim3(kThreads), 0, s, tris, (const int32_t*)deg, slots,
                       (const uint32_t*)head, (const uint32_t*)next, (const int32_t*)heavy, inc, col /* not yet written */, row_len, bnd,
                       dinfo);
  }
  if (n_vertices > 0)
    hipLaunchKernelGGL(k_rows_count, dim3(xcd_blocks(L.nblk)), dim3(kThreads), 0, s, tris, n_vertices,
                       (const int32_t*)deg, (const int32_t*)slots, row_len, bnd, bsum, part);
  hipLaunchKernelGGL(k_top_scan, dim3(1), dim3(kTop), 0, s, bsum, L.nblk, row_off + n_vertices, slice_off + L.nsl);
  if (n_vertices > 0)
    hipLaunchKernelGGL(k_rows_fill, dim3(xcd_blocks((n_vertices + 63) / 64)), dim3(64), 0, s, v, tris, n_vertices, (const int32_t*)deg,
                       (const int32_t*)slots, (const int32_t*)row_len, (const longlong2*)bsum, L.nsl, L.cap, row_off,
                       slice_off, col, val, col_s, val_s, mass, part);
  if (n_triangles > 0)
    hipLaunchKernelGGL(k_heavy_fill, hgrid, dim3(kThreads), 0, s, v, tris, (const int32_t*)deg, (const int32_t*)slots,
                       (const int32_t*)heavy, (const int32_t*)inc, (const int64_t*)row_off, (const int64_t*)slice_off,
                       L.nsl, L.cap, col, val, col_s, val_s, mass, part, (const Info*)dinfo);
  hipLaunchKernelGGL(k_finish, dim3(1), dim3(kParts), 0, s, (const Part*)part, (const int64_t*)row_off + n_vertices,
                     dinfo);
  if (hipGetLastError() != hipSuccess) return SBMT_E_DEVICE;
  Info hi;
  if (hipMemcpyAsync(&hi, dinfo, sizeof(Info), hipMemcpyDeviceToHost, s) != hipSuccess) return SBMT_E_DEVICE;
  if (hipStreamSynchronize(s) != hipSuccess) return SBMT_E_DEVICE;
  info->n_vertices = n_vertices;
  info->nnz = hi.nnz;
  info->n_boundary = hi.n_boundary;
  info->n_invalid = hi.n_invalid;
  // no finite mass seen (no vertex, or NaN masses only): +inf like an empty minimum
  info->min_mass = hi.min_mass_key == ~0ull ? INFINITY : host_key_value(hi.min_mass_key);
  info->lambda_bound = hi.lambda_key == 0ull ? 0.0 : host_key_value(hi.lambda_key);
  return SBMT_OK;
}

sbmt_status sbmt_laplacian_apply(sbmt_handle h, const void* workspace, size_t ws_bytes, int64_t n_vertices,
                                 int64_t n_triangles, const double* u, double* y, void* stream) {
  if (!h || !sizes_ok(n_vertices, n_triangles) || (n_vertices > 0 && (!u || !y))) return SBMT_E_INVALID_ARG;
  const Layout L = layout(n_vertices, n_triangles);
  if (!workspace || ws_bytes < L.total) return SBMT_E_WORKSPACE;
  if (n_vertices == 0) return SBMT_OK;
  hipLaunchKernelGGL(k_apply, dim3(grid_for(n_vertices)), dim3(kThreads), 0, (hipStream_t)stream,
                     op_of((const char*)workspace, L), n_vertices, u, y);
  return hipGetLastError() == hipSuccess ? SBMT_OK : SBMT_E_DEVICE;
}

sbmt_status sbmt_heat_init(sbmt_handle h, const void* workspace, size_t ws_bytes, const double* verts,
                           int64_t n_vertices, int64_t n_triangles, double x0, double y0, double sigma, double amp,
                           double* u, void* stream) {
  if (!h || !sizes_ok(n_vertices, n_triangles) || (n_vertices > 0 && (!u || !verts)) || !(sigma > 0.0))
    return SBMT_E_INVALID_ARG;
  const Layout L = layout(n_vertices, n_triangles);
  if (!workspace || ws_bytes < L.total) return SBMT_E_WORKSPACE;
  if (n_vertices == 0) return SBMT_OK;
  const char* w = (const char*)workspace;
  hipLaunchKernelGGL(k_heat_init, dim3(grid_for(n_vertices)), dim3(kThreads), 0, (hipStream_t)stream,
                     (const double2*)verts, (const uint8_t*)(w + L.bnd), n_vertices, x0, y0, sigma, amp, u);
  return hipGetLastError() == hipSuccess ? SBMT_OK : SBMT_E_DEVICE;
}

sbmt_status sbmt_heat_steps(sbmt_handle h, const void* workspace, size_t ws_bytes, int64_t n_vertices,
                            int64_t n_triangles, double alpha, double dt, int32_t steps, double* u, double* u_tmp,
                            void* stream) {
  if (!h || !sizes_ok(n_vertices, n_triangles) || steps < 0 || (n_vertices > 0 && (!u || !u_tmp)) || u == u_tmp)
    return SBMT_E_INVALID_ARG;
  const Layout L = layout(n_vertices, n_triangles);
  if (!workspace || ws_bytes < L.total) return SBMT_E_WORKSPACE;
  if (n_vertices == 0 || steps == 0) return SBMT_OK;
  hipStream_t s = (hipStream_t)stream;
  const double dt_alpha = dt * alpha;
  const Op op = op_of((const char*)workspace, L);
  double* a = u;
  double* b = u_tmp;
  for (int32_t k = 0; k < steps; ++k) {
    hipLaunchKernelGGL(k_heat_step, dim3(grid_for(n_vertices)), dim3(kThreads), 0, s, op, n_vertices, dt_alpha,
                       (const double*)a, b);
    double* t = a;
    a = b;
    b = t;
  }
  if (a != u) hipLaunchKernelGGL(k_copy, dim3(grid_for(n_vertices)), dim3(kThreads), 0, s, (const double*)a, n_vertices, u);
  return hipGetLastError() == hipSuccess ? SBMT_OK : SBMT_E_DEVICE;
}

}  // extern "C"
