// Dual-mesh mapper (Sec. 3): visual vertices embedded on the simulation
// surface by nearest triangle, barycentric coordinates of the plane
// projection and a signed normal offset (Eqs. (bary_proj), (decomp),
// (gram)); per frame they follow the deformed triangles (Eq. (bary_interp)).
//
// Embedding, few triangles or no scratch memory (k_embed): one thread per
// visual vertex, FP64.  Each block streams the simulation triangles through
// LDS in tiles of 256 (vertex, edges, unit normal, Gram entries and
// inverses, bounding sphere), and every thread scans them in ascending order
// keeping the strict minimum, so ties go to the smaller index.  A triangle
// whose bounding sphere lies farther than the best distance so far is
// skipped without the exact test (it cannot win).
//
// Embedding, with scratch memory (k_tree_query): every vertex against every
// sphere is what bounds k_embed (13.6 ms for 655362 vertices on 20480
// triangles).  The triangles are put in the order of the cells of a 64^3 grid
// along a Hilbert curve (a counting sort: histogram, scan, scatter) and a
// tree of boxes with eight children per node is laid over them (leaves of
// eight).  Eight lanes take one vertex through it, a lane per child or
// triangle, nearest child first; a few thousand vertices already fill the
// device.  The order inside a cell is whatever the atomics gave,
// which the result does not depend on: the smallest (distance, index) wins.
//
// k_update: one thread per visual vertex; three gathered simulation
// vertices (L2-resident for a surface of ~10^4-10^5 vertices), 32 B of
// mapping read and 12 B written per vertex in float.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/gmcp.h"
#include "../../include/gmcp_dualmesh.h"

namespace {

constexpr int kEmbedThreads = 256;

struct TriL {
  double a[3], e1[3], e2[3], n[3];
  double g11, g12, g22, inv_det, ig11, ig22, ie3;
  double c[3], rho;
};

__device__ inline double dot3(const double *x, const double *y) { return x[0] * y[0] + x[1] * y[1] + x[2] * y[2]; }

// squared distance from p to triangle T (nearest point of the triangle)
__device__ inline double tri_dist2(const double p[3], const TriL &T) {
  double d[3] = {p[0] - T.a[0], p[1] - T.a[1], p[2] - T.a[2]};
  const double r1 = dot3(d, T.e1), r2 = dot3(d, T.e2);
  const double v = (T.g22 * r1 - T.g12 * r2) * T.inv_det;
  const double w = (T.g11 * r2 - T.g12 * r1) * T.inv_det;
  if (v >= 0.0 && w >= 0.0 && v + w <= 1.0) {
    const double dn = dot3(d, T.n);
    return dn * dn;
  }
  // nearest point on the boundary: edges a->b, a->c, b->c
  double best;
  {
    const double t = fmin(fmax(r1 * T.ig11, 0.0), 1.0);
    const double q0 = d[0] - t * T.e1[0], q1 = d[1] - t * T.e1[1], q2 = d[2] - t * T.e1[2];
    best = q0 * q0 + q1 * q1 + q2 * q2;
  }
  {
    const double t = fmin(fmax(r2 * T.ig22, 0.0), 1.0);
    const double q0 = d[0] - t * T.e2[0], q1 = d[1] - t * T.e2[1], q2 = d[2] - t * T.e2[2];
    best = fmin(best, q0 * q0 + q1 * q1 + q2 * q2);
  }
  {
    const double db[3] = {d[0] - T.e1[0], d[1] - T.e1[1], d[2] - T.e1[2]};
    const double e3[3] = {T.e2[0] - T.e1[0], T.e2[1] - T.e1[1], T.e2[2] - T.e1[2]};
    const double t = fmin(fmax(dot3(db, e3) * T.ie3, 0.0), 1.0);
    const double q0 = db[0] - t * e3[0], q1 = db[1] - t * e3[1], q2 = db[2] - t * e3[2];
    best = fmin(best, q0 * q0 + q1 * q1 + q2 * q2);
  }
  return best;
}

__device__ inline void load_tri(const double *__restrict__ V, const int32_t *__restrict__ F, int64_t t, double a[3],
                                double b[3], double c[3]) {
  for (int k = 0; k < 3; ++k) {
    a[k] = V[(int64_t)F[t * 3 + 0] * 3 + k];
    b[k] = V[(int64_t)F[t * 3 + 1] * 3 + k];
    c[k] = V[(int64_t)F[t * 3 + 2] * 3 + k];
  }
}

// whether two edges span an area.  Not fused: for equal edges (a repeated
// vertex) a fused e1y e2z - e1z e2y leaves its rounding, not zero.
__device__ inline bool spans_area(const double e1[3], const double e2[3]) {
#pragma clang fp contract(off)
  const double x = e1[1] * e2[2], x2 = e1[2] * e2[1], y = e1[2] * e2[0], y2 = e1[0] * e2[2], z = e1[0] * e2[1],
               z2 = e1[1] * e2[0];
  return x != x2 || y != y2 || z != z2;
}

// false for a triangle of zero or non-finite area (never chosen)
__device__ inline bool make_tri(const double a[3], const double b[3], const double c[3], TriL &T) {
  double e1[3], e2[3];
  for (int k = 0; k < 3; ++k) {
    e1[k] = b[k] - a[k];
    e2[k] = c[k] - a[k];
  }
  const double nx = e1[1] * e2[2] - e1[2] * e2[1], ny = e1[2] * e2[0] - e1[0] * e2[2],
               nz = e1[0] * e2[1] - e1[1] * e2[0];
  const double nn = nx * nx + ny * ny + nz * nz;  // = Gram determinant
  const bool ok = nn > 0.0 && isfinite(nn) && spans_area(e1, e2);
  const double inv_n = ok ? 1.0 / sqrt(nn) : 0.0;
  for (int k = 0; k < 3; ++k) {
    T.a[k] = a[k];
    T.e1[k] = e1[k];
    T.e2[k] = e2[k];
    T.c[k] = (a[k] + b[k] + c[k]) * (1.0 / 3.0);
  }
  T.n[0] = nx * inv_n;
  T.n[1] = ny * inv_n;
  T.n[2] = nz * inv_n;
  T.g11 = dot3(e1, e1);
  T.g12 = dot3(e1, e2);
  T.g22 = dot3(e2, e2);
  T.inv_det = ok ? 1.0 / (T.g11 * T.g22 - T.g12 * T.g12) : 0.0;
  const double e3[3] = {c[0] - b[0], c[1] - b[1], c[2] - b[2]};
  T.ig11 = ok ? 1.0 / T.g11 : 0.0;
  T.ig22 = ok ? 1.0 / T.g22 : 0.0;
  T.ie3 = ok ? 1.0 / dot3(e3, e3) : 0.0;
  double r = 0.0;
  for (int k = 0; k < 3; ++k) {
    const double *q = k == 0 ? a : (k == 1 ? b : c);
    const double dx = q[0] - T.c[0], dy = q[1] - T.c[1], dz = q[2] - T.c[2];
    r = fmax(r, dx * dx + dy * dy + dz * dz);
  }
  T.rho = sqrt(r);
  return ok;
}

// the mapping of vertex i at p on triangle bt (-1: none), Eqs. (decomp), (gram)
__device__ inline void write_map(int64_t i, const double p[3], double best, int32_t bt, const double *__restrict__ V,
                                 const int32_t *__restrict__ F, int32_t *__restrict__ tri, double *__restrict__ bary,
                                 double *__restrict__ delta, double *__restrict__ dist2) {
  tri[i] = bt;
  if (dist2) dist2[i] = best;
  if (bt < 0) {
    for (int k = 0; k < 3; ++k) bary[i * 3 + k] = NAN;
    delta[i] = NAN;
    return;
  }
  // Eqs. (decomp), (gram) on the chosen triangle
  double a[3], e1[3], e2[3], d[3];
  for (int k = 0; k < 3; ++k) {
    a[k] = V[(int64_t)F[(int64_t)bt * 3 + 0] * 3 + k];
    e1[k] = V[(int64_t)F[(int64_t)bt * 3 + 1] * 3 + k] - a[k];
    e2[k] = V[(int64_t)F[(int64_t)bt * 3 + 2] * 3 + k] - a[k];
    d[k] = p[k] - a[k];
  }
  const double g11 = dot3(e1, e1), g12 = dot3(e1, e2), g22 = dot3(e2, e2);
  const double r1 = dot3(d, e1), r2 = dot3(d, e2);
  const double det = g11 * g22 - g12 * g12;
  const double v = (g22 * r1 - g12 * r2) / det, w = (g11 * r2 - g12 * r1) / det;
  const double n[3] = {e1[1] * e2[2] - e1[2] * e2[1], e1[2] * e2[0] - e1[0] * e2[2], e1[0] * e2[1] - e1[1] * e2[0]};
  const double nl = sqrt(dot3(n, n));
  bary[i * 3 + 0] = 1.0 - v - w;
  bary[i * 3 + 1] = v;
  bary[i * 3 + 2] = w;
  delta[i] = dot3(d, n) / nl;
}

__global__ __launch_bounds__(kEmbedThreads) void k_embed(const double *__restrict__ P, int64_t N,
                                                         const double *__restrict__ V, const int32_t *__restrict__ F,
                                                         int64_t nT, int32_t *__restrict__ tri,
                                                         double *__restrict__ bary, double *__restrict__ delta,
                                                         double *__restrict__ dist2) {
  __shared__ TriL tl[kEmbedThreads];
  __shared__ int valid[kEmbedThreads];
  const int64_t i = (int64_t)blockIdx.x * kEmbedThreads + threadIdx.x;
  const bool live = i < N;
  double p[3] = {0.0, 0.0, 0.0};
  if (live)
    for (int k = 0; k < 3; ++k) p[k] = P[i * 3 + k];
  double best = INFINITY;
  int32_t bt = -1;
  for (int64_t t0 = 0; t0 < nT; t0 += kEmbedThreads) {
    __syncthreads();
    const int64_t t = t0 + threadIdx.x;
    int ok = 0;
    if (t < nT) {
      double a[3], b[3], c[3];
      load_tri(V, F, t, a, b, c);
      ok = make_tri(a, b, c, tl[threadIdx.x]);
    }
    valid[threadIdx.x] = ok;
    __syncthreads();
    if (!live) continue;
    const int cnt = (int)((nT - t0) < kEmbedThreads ? (nT - t0) : kEmbedThreads);
    double sb = sqrt(best);
    for (int j = 0; j < cnt; ++j) {
      if (!valid[j]) continue;
      const TriL &T = tl[j];
      const double dx = p[0] - T.c[0], dy = p[1] - T.c[1], dz = p[2] - T.c[2];
      const double reach = (sb + T.rho) * (1.0 + 1e-12);
      if (dx * dx + dy * dy + dz * dz > reach * reach) continue;  // every point of T is farther than best
      const double d2 = tri_dist2(p, T);
      if (d2 < best) {
        best = d2;
        bt = (int32_t)(t0 + j);
        sb = sqrt(best);
      }
    }
  }
  if (!live) return;
  write_map(i, p, best, bt, V, F, tri, bary, delta, dist2);
}

// ------------------------------------------------------------------ tree
constexpr int kGridBits = 6;                          // 64^3 cells, numbered along a Hilbert curve
constexpr int kCells = 1 << (3 * kGridBits);
constexpr int kStart = kCells + 4;                    // the scan's total after the last cell
// Fewest vertices that are put in the curve's order too (vertices listed in
// no spatial order then share nodes and triangles in the caches): the sort
// costs 50 us at 655362 and the walk drops from 583 to 487 us; at 131072
// they are even.
constexpr int64_t kSortPoints = 131072;
constexpr int kScanCells = 16384;                     // cells per block of the scan
constexpr int kLeaf = 8, kFan = 8;                    // triangles per leaf, children per node
constexpr int kMaxLevels = 8;                         // leaves, then eight times fewer per level, to one node's children
constexpr int64_t kTreeMax = int64_t(1) << 27;        // triangles: 8^8 leaves' worth
constexpr int64_t kTreePoints = int64_t(1) << 30;
constexpr int kNodeThreads = kLeaf * kFan * kFan;     // sorted triangles per block of k_tree_nodes
constexpr int kWaveT = 64;

struct Box {  // float, rounded outwards
  float lo[3], hi[3];
};

struct TreeDev {
  uint32_t *bounds;        // [6] the surface's box (ordered float bits)
  int32_t *hist, *start;   // [2][cells], [2][cells + 4]: triangles, vertices
  int32_t *cell, *rank;    // [nT + N] cell (-1: not taken) and place in it
  int32_t *pid;            // [N] vertex at each sorted place, null: vertices are taken in their own order
  int32_t *id;             // [nT] triangle at each sorted place
  TriL *tl;                // [nT] sorted
  Box *node[kMaxLevels];   // [cnt up to a multiple of eight], empty boxes after the last
  int32_t cnt[kMaxLevels];
  int top;                 // level the walk starts at (at least 2), of at most eight nodes
};

size_t tree_plan(int64_t N, int64_t nT, char *base, TreeDev *out) {
  size_t off = 0;
  auto take = [&](size_t bytes) {
    off = (off + 255) & ~size_t(255);
    char *p = base ? base + off : nullptr;
    off += bytes;
    return p;
  };
  TreeDev t{};
  t.bounds = (uint32_t *)take(6 * sizeof(uint32_t));
  const int64_t sorted = N >= kSortPoints ? N : 0;
  t.hist = (int32_t *)take(sizeof(int32_t) * 2 * kCells);
  t.start = (int32_t *)take(sizeof(int32_t) * 2 * kStart);
  t.cell = (int32_t *)take(sizeof(int32_t) * (size_t)(nT + sorted));
  t.rank = (int32_t *)take(sizeof(int32_t) * (size_t)(nT + sorted));
  if (sorted) t.pid = (int32_t *)take(sizeof(int32_t) * (size_t)sorted);
  t.id = (int32_t *)take(sizeof(int32_t) * (size_t)nT);
  t.tl = (TriL *)take(sizeof(TriL) * (size_t)nT);
  int64_t c = (nT + kLeaf - 1) / kLeaf;
  for (t.top = 0; t.top < kMaxLevels; ++t.top) {
    t.cnt[t.top] = (int32_t)c;
    // the node kernel's blocks write 64 leaves and 8 level-1 nodes each
    const int64_t unit = t.top == 0 ? kFan * kFan : kFan;
    t.node[t.top] = (Box *)take(sizeof(Box) * (size_t)((c + unit - 1) / unit * unit));
    if (t.top >= 2 && c <= kFan) break;
    c = (c + kFan - 1) / kFan;
  }
  if (out) *out = t;
  return off + 256;
}

__device__ inline uint32_t ordered(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline float unordered(uint32_t u) { return __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u); }

__global__ __launch_bounds__(256) void k_tree_clear(TreeDev t) {
  const int i = blockIdx.x * 256 + threadIdx.x;  // four cells each
  reinterpret_cast<int4 *>(t.hist)[i] = make_int4(0, 0, 0, 0);
  if (i < 6) t.bounds[i] = i < 3 ? 0xffffffffu : 0u;
}

// the valid triangles' box, in float: it only sets the order of the sort.
// Few, large blocks: every block's six atomics meet at the same words.
constexpr int kBoundThreads = 1024;
__global__ __launch_bounds__(kBoundThreads) void k_tree_bounds(const double *__restrict__ V,
                                                               const int32_t *__restrict__ F, int64_t nT, TreeDev t) {
  __shared__ uint32_t wlo[kBoundThreads / kWaveT][3], whi[kBoundThreads / kWaveT][3];
  uint32_t lo[3] = {0xffffffffu, 0xffffffffu, 0xffffffffu}, hi[3] = {0u, 0u, 0u};
  for (int64_t i = (int64_t)blockIdx.x * kBoundThreads + threadIdx.x; i < nT;
       i += (int64_t)gridDim.x * kBoundThreads) {
    double a[3], b[3], c[3];
    TriL T;
    load_tri(V, F, i, a, b, c);
    if (!make_tri(a, b, c, T)) continue;
    for (int k = 0; k < 3; ++k) {
      const uint32_t u = ordered((float)T.c[k]);
      lo[k] = min(lo[k], u);
      hi[k] = max(hi[k], u);
    }
  }
  for (int k = 0; k < 3; ++k)
    for (int o = kWaveT / 2; o > 0; o >>= 1) {
      lo[k] = min(lo[k], (uint32_t)__shfl_xor((int)lo[k], o, kWaveT));
      hi[k] = max(hi[k], (uint32_t)__shfl_xor((int)hi[k], o, kWaveT));
    }
  if (threadIdx.x % kWaveT == 0)
    for (int k = 0; k < 3; ++k) {
      wlo[threadIdx.x / kWaveT][k] = lo[k];
      whi[threadIdx.x / kWaveT][k] = hi[k];
    }
  __syncthreads();
  if (threadIdx.x < 3) {
    const int k = threadIdx.x;
    uint32_t l = 0xffffffffu, h = 0u;
    for (int w = 0; w < kBoundThreads / kWaveT; ++w) {
      l = min(l, wlo[w][k]);
      h = max(h, whi[w][k]);
    }
    atomicMin(&t.bounds[k], l);
    atomicMax(&t.bounds[3 + k], h);
  }
}

// Cell of a point (clamped to the surface's box), numbered along the Hilbert
// curve by Skilling's transform ("Programming the Hilbert curve", AIP Conf.
// Proc. 707, 2004): neighbours in that order span less than in Morton order,
// so the boxes over eight of them are tighter.
__device__ inline int curve_cell(const double p[3], const uint32_t *__restrict__ bounds) {
  uint32_t x[3];
  for (int k = 0; k < 3; ++k) {
    const float lo = unordered(bounds[k]), hi = unordered(bounds[3 + k]);
    const float f = ((float)p[k] - lo) / (hi - lo) * (float)(1 << kGridBits);
    // NaN (a flat box): 0
    x[k] = f > 0.0f ? min((uint32_t)fminf(f, (float)(1 << kGridBits)), (1u << kGridBits) - 1) : 0u;
  }
#pragma unroll
  for (uint32_t q = 1u << (kGridBits - 1); q > 1; q >>= 1) {
    const uint32_t m = q - 1;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if (x[k] & q) {
        x[0] ^= m;
      } else {
        const uint32_t t = (x[0] ^ x[k]) & m;
        x[0] ^= t;
        x[k] ^= t;
      }
    }
  }
  x[1] ^= x[0];
  x[2] ^= x[1];
  uint32_t t = 0;
#pragma unroll
  for (uint32_t q = 1u << (kGridBits - 1); q > 1; q >>= 1)
    if (x[2] & q) t ^= q - 1;
  int cell = 0;
#pragma unroll
  for (int b = kGridBits - 1; b >= 0; --b)
    for (int k = 0; k < 3; ++k) cell = (cell << 1) | (int)(((x[k] ^ t) >> b) & 1u);
  return cell;
}

// item i: triangle i, or vertex i - nT
__global__ __launch_bounds__(256) void k_tree_count(const double *__restrict__ P, int64_t n,
                                                    const double *__restrict__ V, const int32_t *__restrict__ F,
                                                    int64_t nT, TreeDev t) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  int cell = -1;
  if (i >= nT) {
    double p[3];
    for (int k = 0; k < 3; ++k) p[k] = P[(i - nT) * 3 + k];
    cell = curve_cell(p, t.bounds) + kCells;
  } else {
    double a[3], b[3], c[3];
    TriL T;
    load_tri(V, F, i, a, b, c);
    if (make_tri(a, b, c, T)) cell = curve_cell(T.c, t.bounds);
  }
  t.cell[i] = cell;
  if (cell >= 0) t.rank[i] = atomicAdd(&t.hist[cell], 1);
}

// exclusive scan of the histogram: a block sums the cells before its own (no
// other block to wait for), then scans its own
__global__ __launch_bounds__(1024) void k_tree_scan(TreeDev t) {
  constexpr int kPer = kScanCells / 1024;
  __shared__ int wsum[1024 / kWaveT], before[1024 / kWaveT];
  const int4 *in4 = reinterpret_cast<const int4 *>(t.hist + (size_t)blockIdx.y * kCells);
  const int lane = threadIdx.x % kWaveT, w = threadIdx.x / kWaveT;
  const int first = blockIdx.x * (kScanCells / 4);
  int pre = 0;
#pragma unroll 4
  for (int k = threadIdx.x; k < first; k += 1024) {
    const int4 v = in4[k];
    pre += v.x + v.y + v.z + v.w;
  }
  int4 v[kPer / 4];
  int sum = 0;
#pragma unroll
  for (int k = 0; k < kPer / 4; ++k) {
    v[k] = in4[first + threadIdx.x * (kPer / 4) + k];
    sum += v[k].x + v[k].y + v[k].z + v[k].w;
  }
  int inc = sum;
  for (int o = 1; o < kWaveT; o <<= 1) {
    const int up = __shfl_up(inc, o, kWaveT);
    if (lane >= o) inc += up;
  }
  for (int o = kWaveT / 2; o > 0; o >>= 1) pre += __shfl_xor(pre, o, kWaveT);
  if (lane == kWaveT - 1) {
    wsum[w] = inc;
    before[w] = pre;
  }
  __syncthreads();
  int run = inc - sum;
  for (int k = 0; k < 1024 / kWaveT; ++k) run += before[k] + (k < w ? wsum[k] : 0);
  int4 *out4 = reinterpret_cast<int4 *>(t.start + (size_t)blockIdx.y * kStart) + first + threadIdx.x * (kPer / 4);
#pragma unroll
  for (int k = 0; k < kPer / 4; ++k) {
    int4 o;
    o.x = run;
    o.y = o.x + v[k].x;
    o.z = o.y + v[k].y;
    o.w = o.z + v[k].z;
    run = o.w + v[k].w;
    out4[k] = o;
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 1023) t.start[(size_t)blockIdx.y * kStart + kCells] = run;
}

__global__ __launch_bounds__(256) void k_tree_place(int64_t n, const double *__restrict__ V,
                                                    const int32_t *__restrict__ F, int64_t nT, TreeDev t) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int cell = t.cell[i];
  if (cell < 0) return;
  const int64_t at = (int64_t)t.start[i >= nT ? cell - kCells + kStart : cell] + t.rank[i];
  if (i >= nT) {
    t.pid[at] = (int32_t)(i - nT);
    return;
  }
  double a[3], b[3], c[3];
  TriL T;
  load_tri(V, F, i, a, b, c);
  make_tri(a, b, c, T);
  t.tl[at] = T;
  t.id[at] = (int32_t)i;
}

__device__ inline Box empty_box() {
  Box b;
  for (int k = 0; k < 3; ++k) {
    b.lo[k] = INFINITY;
    b.hi[k] = -INFINITY;
  }
  return b;
}

__device__ inline void box_add(Box &b, const Box &o) {
  for (int k = 0; k < 3; ++k) {
    b.lo[k] = fminf(b.lo[k], o.lo[k]);
    b.hi[k] = fmaxf(b.hi[k], o.hi[k]);
  }
}

__device__ inline void box_merge(Box &b, int o) {
  for (int k = 0; k < 3; ++k) {
    b.lo[k] = fminf(b.lo[k], __shfl_xor(b.lo[k], o, kWaveT));
    b.hi[k] = fmaxf(b.hi[k], __shfl_xor(b.hi[k], o, kWaveT));
  }
}

// the three lowest levels: a thread per sorted triangle, eight lanes per
// leaf, a wave per level-1 node, a block per level-2 node.  A box is rounded
// outwards by more than the float and the distance computations round, so
// a pruned triangle's computed distance cannot come out below the best one.
__global__ __launch_bounds__(kNodeThreads) void k_tree_nodes(TreeDev t) {
  __shared__ Box wb[kNodeThreads / kWaveT];
  const int64_t i = (int64_t)blockIdx.x * kNodeThreads + threadIdx.x;
  const int lane = threadIdx.x % kWaveT, w = threadIdx.x / kWaveT;
  Box b = empty_box();
  if (i < t.start[kCells]) {
    const TriL &T = t.tl[i];
    float m = 0.0f;
    for (int k = 0; k < 3; ++k) {
      const double v0 = T.a[k], v1 = v0 + T.e1[k], v2 = v0 + T.e2[k];
      // (beyond float: the largest float on the inner side keeps the box a bound)
      b.lo[k] = fminf((float)fmin(v0, fmin(v1, v2)), 3.4e38f);
      b.hi[k] = fmaxf((float)fmax(v0, fmax(v1, v2)), -3.4e38f);
      m = fmaxf(m, fmaxf(fabsf(b.lo[k]), fabsf(b.hi[k])));
    }
    m = m * 2.5e-7f + 1.2e-38f;
    for (int k = 0; k < 3; ++k) {
      b.lo[k] -= m;
      b.hi[k] += m;
    }
  }
  for (int o = 1; o < kLeaf; o <<= 1) box_merge(b, o);
  if (lane % kLeaf == 0) t.node[0][i / kLeaf] = b;  // 64 per block: within the rounded count
  for (int o = kLeaf; o < kWaveT; o <<= 1) box_merge(b, o);
  if (lane == 0) {
    wb[w] = b;
    t.node[1][i / kWaveT] = b;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < kNodeThreads / kWaveT; ++k) box_add(b, wb[k]);
    t.node[2][blockIdx.x] = b;
    if (blockIdx.x == gridDim.x - 1)
      for (int k = gridDim.x; k % kFan; ++k) t.node[2][k] = empty_box();
  }
}

// one level above the third
__global__ __launch_bounds__(256) void k_tree_up(TreeDev t, int level) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= (t.cnt[level] + kFan - 1) / kFan * kFan) return;
  Box b = empty_box();
  const int c1 = min(kFan * (i + 1), t.cnt[level - 1]);
  for (int c = kFan * i; c < c1; ++c) box_add(b, t.node[level - 1][c]);
  t.node[level][i] = b;
}

// Squared distance from [pl, ph] (a point's coordinates rounded down and up)
// to a box, in float: at most 1e-6 above that of the point to what the box
// bounds.  (In double this test was half of the walk's instructions.)
__device__ inline float box_dist2(const float pl[3], const float ph[3], const Box &b) {
  float s = 0.0f;
  for (int k = 0; k < 3; ++k) {
    const float d = fmaxf(fmaxf(b.lo[k] - ph[k], pl[k] - b.hi[k]), 0.0f);
    s += d * d;
  }
  return s;
}

// lane moves within groups of eight lanes: 1 and 2 lanes apart, and the mirror
template <int CTRL>
__device__ inline uint32_t move8(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
}
constexpr int kQuad1 = 0xB1, kQuad2 = 0x4E, kHalfMirror = 0x141;
template <int CTRL>
__device__ inline void min8(uint32_t &v) {
  v = min(v, move8<CTRL>(v));
}
// the smaller (d, id) of the lane and its partner
template <int CTRL>
__device__ inline void best8(double &d, int32_t &id) {
  const double od = __hiloint2double((int)move8<CTRL>((uint32_t)__double2hiint(d)),
                                     (int)move8<CTRL>((uint32_t)__double2loint(d)));
  const int32_t oid = (int32_t)move8<CTRL>((uint32_t)id);
  if (od < d || (od == d && oid < id)) {
    d = od;
    id = oid;
  }
}

// Bound by the latency of its gathers: a vertex takes about 18 steps and 5
// leaves (28 and 8 for the slowest of a wave's eight), each a dependent load.
// 655362 vertices on 20480 triangles: 400 us (460 us the whole embedding,
// 13.6 ms by the scan); 2562 vertices: 93 us (3.6 ms).  A wave walking with
// 64 sorted vertices together, nodes and triangles by scalar loads, took
// 331 us there but 890 us for the 2562 vertices.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8))) void k_tree_query(
    const double *__restrict__ P, int64_t N, const double *__restrict__ V, const int32_t *__restrict__ F,
                                                    TreeDev t, int32_t *__restrict__ tri, double *__restrict__ bary,
                                                    double *__restrict__ delta, double *__restrict__ dist2) {
  __shared__ float kept[kMaxLevels - 1][256];  // d of the levels above: kept[l] is level l + 1's
  const int64_t s = ((int64_t)blockIdx.x * 256 + threadIdx.x) / kFan;
  const int c = threadIdx.x % kFan;
  const bool in = s < N;
  const int64_t i = in && t.pid ? t.pid[s] : s;
  double p[3] = {0.0, 0.0, 0.0};
  if (in)
    for (int k = 0; k < 3; ++k) p[k] = P[i * 3 + k];
  const bool live = in && isfinite(p[0]) && isfinite(p[1]) && isfinite(p[2]);
  const int n_tri = t.start[kCells];
  double best = live ? INFINITY : -INFINITY, sb = best;  // a vertex that is not finite opens nothing
  int32_t bt = -1;
  // best, bt and the walk's state are the same in the eight lanes of a vertex
  float pl[3], ph[3];
  for (int k = 0; k < 3; ++k) {
    const float f = fminf(fmaxf((float)p[k], -3.4e38f), 3.4e38f), e = fabsf(f) * 1.2e-7f + 1.2e-38f;
    pl[k] = f - e;
    ph[k] = f + e;
  }
  float bound = (float)best;
  // d: distance of the lane's child of the current node, NaN once visited
  int level = t.top, base = 0;
  float d = box_dist2(pl, ph, t.node[level][c]);
  for (;;) {
    // nearest open child: its distance's bits with the child in the low three
    uint32_t key = d <= bound ? (__float_as_uint(d) & ~7u) | (uint32_t)c : 0xffffffffu;
    min8<kQuad1>(key);
    min8<kQuad2>(key);
    min8<kHalfMirror>(key);
    if (key == 0xffffffffu) {
      if (level == t.top) break;
      base = base / kFan / kFan * kFan;
      d = kept[level++][threadIdx.x];
      continue;
    }
    if ((int)(key & 7u) == c) d = NAN;
    const int at = base + (int)(key & 7u);
    if (level > 0) {
      kept[--level][threadIdx.x] = d;
      base = kFan * at;
      d = box_dist2(pl, ph, t.node[level][base + c]);
      continue;
    }
    // a leaf: a triangle per lane
    const int j = kLeaf * at + c;
    double d2 = INFINITY;
    int32_t id = INT32_MAX;
    if (j < n_tri) {
      const TriL &T = t.tl[j];
      const double dx = p[0] - T.c[0], dy = p[1] - T.c[1], dz = p[2] - T.c[2];
      const double reach = (sb + T.rho) * (1.0 + 1e-12);
      if (!(dx * dx + dy * dy + dz * dz > reach * reach)) {  // else every point of T is farther than best
        d2 = tri_dist2(p, T);
        id = t.id[j];
        if (!(d2 < INFINITY)) {  // overflow, NaN: never chosen
          d2 = INFINITY;
          id = INT32_MAX;
        }
      }
    }
    best8<kQuad1>(d2, id);
    best8<kQuad2>(d2, id);
    best8<kHalfMirror>(d2, id);
    if (d2 < best || (d2 == best && id < bt)) {
      best = d2;
      bt = id;
      sb = sqrt(best);
      bound = (float)best * 1.000002f;
    }
  }
  if (in && c == 0) write_map(i, p, bt < 0 ? INFINITY : best, bt, V, F, tri, bary, delta, dist2);
}

template <typename R>
__device__ inline R rsqrt_r(R x);
template <>
__device__ inline float rsqrt_r<float>(float x) {
  return rsqrtf(x);
}
template <>
__device__ inline double rsqrt_r<double>(double x) {
  return 1.0 / sqrt(x);
}

template <typename R>
__global__ __launch_bounds__(256) void k_update(const R *__restrict__ Vd, const int32_t *__restrict__ F,
                                                const int32_t *__restrict__ tri, const R *__restrict__ bary,
                                                const R *__restrict__ delta, int64_t N, R *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= N) return;
  const int64_t t = tri[i];
  const int64_t i0 = F[t * 3 + 0], i1 = F[t * 3 + 1], i2 = F[t * 3 + 2];
  const R ax = Vd[i0 * 3], ay = Vd[i0 * 3 + 1], az = Vd[i0 * 3 + 2];
  const R bx = Vd[i1 * 3], by = Vd[i1 * 3 + 1], bz = Vd[i1 * 3 + 2];
  const R cx = Vd[i2 * 3], cy = Vd[i2 * 3 + 1], cz = Vd[i2 * 3 + 2];
  const R e1x = bx - ax, e1y = by - ay, e1z = bz - az;
  const R e2x = cx - ax, e2y = cy - ay, e2z = cz - az;
  const R nx = e1y * e2z - e1z * e2y, ny = e1z * e2x - e1x * e2z, nz = e1x * e2y - e1y * e2x;
  const R s = delta[i] * rsqrt_r<R>(nx * nx + ny * ny + nz * nz);
  const R u = bary[i * 3], v = bary[i * 3 + 1], w = bary[i * 3 + 2];
  out[i * 3 + 0] = u * ax + v * bx + w * cx + s * nx;
  out[i * 3 + 1] = u * ay + v * by + w * cy + s * ny;
  out[i * 3 + 2] = u * az + v * bz + w * cz + s * nz;
}

// Fewest triangles the tree is used for.  Its eight launches take at least
// 58 us; the scan, a chain of nT sphere tests, takes 90 us at 320 triangles
// and 174 us at 720 (2562 vertices), about as long at 256.
constexpr int64_t kTreeTriangles = 256;

inline unsigned nblocks(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

}  // namespace

extern "C" {

int gmcp_dualmesh_embed(const double *P, int64_t N, const double *V, const int32_t *F, int64_t nT, int32_t *tri,
                        double *bary, double *delta, double *dist2, void *stream) {
  if (N < 0 || nT < 0) return GMCP_E_ARG;
  if (N == 0) return GMCP_OK;
  if (nT == 0 || !P || !V || !F || !tri || !bary || !delta) return GMCP_E_ARG;
  hipLaunchKernelGGL(k_embed, dim3(nblocks(N, kEmbedThreads)), dim3(kEmbedThreads), 0, (hipStream_t)stream, P, N, V,
                     F, nT, tri, bary, delta, dist2);
  return hipGetLastError() == hipSuccess ? GMCP_OK : GMCP_E_HIP;
}

size_t gmcp_dualmesh_embed_work_bytes(int64_t N, int64_t nT) {
  if (N < 0 || nT < kTreeTriangles || N > kTreePoints || nT > kTreeMax) return 0;
  return tree_plan(N, nT, nullptr, nullptr);
}

int gmcp_dualmesh_embed_ws(const double *P, int64_t N, const double *V, const int32_t *F, int64_t nT, int32_t *tri,
                           double *bary, double *delta, double *dist2, void *work, size_t work_bytes, void *stream) {
  const size_t need = gmcp_dualmesh_embed_work_bytes(N, nT);
  if (need == 0 || !work) return gmcp_dualmesh_embed(P, N, V, F, nT, tri, bary, delta, dist2, stream);
  if (work_bytes < need) return GMCP_E_ARG;
  if (N == 0) return GMCP_OK;
  if (!P || !V || !F || !tri || !bary || !delta) return GMCP_E_ARG;
  TreeDev t;
  tree_plan(N, nT, (char *)((reinterpret_cast<uintptr_t>(work) + 255) & ~uintptr_t(255)), &t);
  hipStream_t s = (hipStream_t)stream;
  const int sets = t.pid ? 2 : 1;
  const int64_t items = nT + (t.pid ? N : 0);
  hipLaunchKernelGGL(k_tree_clear, dim3(sets * kCells / 1024), dim3(256), 0, s, t);
  hipLaunchKernelGGL(k_tree_bounds, dim3(std::min(nblocks(nT, kBoundThreads), 64u)), dim3(kBoundThreads), 0, s, V, F,
                     nT, t);
  hipLaunchKernelGGL(k_tree_count, dim3(nblocks(items, 256)), dim3(256), 0, s, P, items, V, F, nT, t);
  hipLaunchKernelGGL(k_tree_scan, dim3(kCells / kScanCells, sets), dim3(1024), 0, s, t);
  hipLaunchKernelGGL(k_tree_place, dim3(nblocks(items, 256)), dim3(256), 0, s, items, V, F, nT, t);
  hipLaunchKernelGGL(k_tree_nodes, dim3(nblocks(nT, kNodeThreads)), dim3(kNodeThreads), 0, s, t);
  for (int l = 3; l <= t.top; ++l)
    hipLaunchKernelGGL(k_tree_up, dim3(nblocks(t.cnt[l] + kFan, 256)), dim3(256), 0, s, t, l);
  hipLaunchKernelGGL(k_tree_query, dim3(nblocks(kFan * N, 256)), dim3(256), 0, s, P, N, V, F, t, tri, bary, delta,
                     dist2);
  return hipGetLastError() == hipSuccess ? GMCP_OK : GMCP_E_HIP;
}

int gmcp_dualmesh_update(const void *Vd, const int32_t *F, const int32_t *tri, const void *bary, const void *delta,
                         int64_t N, void *out, uint32_t flags, void *stream) {
  if (N < 0) return GMCP_E_ARG;
  if (N == 0) return GMCP_OK;
  if (!Vd || !F || !tri || !bary || !delta || !out) return GMCP_E_ARG;
  if (flags & GMCP_F64)
    hipLaunchKernelGGL(k_update<double>, dim3(nblocks(N, 256)), dim3(256), 0, (hipStream_t)stream,
                       (const double *)Vd, F, tri, (const double *)bary, (const double *)delta, N, (double *)out);
  else
    hipLaunchKernelGGL(k_update<float>, dim3(nblocks(N, 256)), dim3(256), 0, (hipStream_t)stream, (const float *)Vd,
                       F, tri, (const float *)bary, (const float *)delta, N, (float *)out);
  return hipGetLastError() == hipSuccess ? GMCP_OK : GMCP_E_HIP;
}

}  // extern "C"
