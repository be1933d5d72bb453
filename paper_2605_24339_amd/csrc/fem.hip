// Implicit-step system around the contact potential: linear-elastic
// tetrahedra, lumped mass, block-Jacobi preconditioned CG on
//   A = M / dt^2 + K + H_contact,
// with Dirichlet vertices held fixed.  Double precision throughout.
//
// K is static: its 3x3 BSR pattern is the vertex adjacency of the tets and
// every block is the sum, in a fixed order, of the element blocks
//   K_e(a,b)_ik = vol (mu (gN_a . gN_b) d_ik + mu gN_b,i gN_a,k + lambda gN_a,i gN_b,k)
// of the tets containing both vertices (gN = gradients of the linear shape
// functions), so the assembled matrix is deterministic.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <map>
#include <new>
#include <vector>

#include "../../include/gmcp_fem.h"
#include "common.h"

namespace {

constexpr int kT = 256;

// K's blocks are kept in slices of 64 rows, lane = row: entry j of a slice
// holds the j-th block of each of its rows, the nine values as nine runs of
// 64 doubles and the columns as one run of 64 ids (-1: the row has fewer
// blocks).  A wave reads an entry with ten coalesced loads; the row-by-row
// form of the same blocks (72 bytes a row apart per lane) streamed at 1.75
// TB/s (40 MB in 22.8 us at 38025 vertices).
constexpr int kSlice = 64;
// waves of a slice's block: wave w takes entries w, w + 4, ...  38025 rows
// are only 594 slices, so the rows' entries are split to have enough loads
// in flight (the four partial sums are added in wave order)
constexpr int kSliceWaves = 4;

struct Sell {
  const int32_t *off;  // [n_slices + 1] first entry of each slice
  const int32_t *col;  // [entries][64]
  const double *val;   // [entries][9][64]
};

struct FemDev {
  int32_t *k_row_ptr, *k_col;  // static BSR pattern of K (V rows)
  int32_t *k_row;              // [nnzb] row of each block
  int32_t *s_off, *s_col;      // sliced form of K (Sell)
  double *s_val;
  int32_t *k_diag;             // [V] the diagonal block's index, -1 if the row is empty
  int32_t *c_off, *c_list;     // per K block: contributions tet*16 + a*4 + b
  double *mass;                // [V] lumped mass
  uint8_t *fixed;              // [V] Dirichlet components: bit d = component d held
  double *X;                   // [V][3] rest positions
  int32_t *tets;               // [n_tet][4]
  double *Pinv;                // [V][9] block-Jacobi inverse
  double *r, *z, *q;           // CG vectors [3V]
  double *p[2];                // search directions of the last two iterations
  double *part_pq, *part_rz, *part_rr;  // partial dot products per block
  double *scal;                // [16] device scalars
  int32_t *done;               // CG has ended: the launches already queued do nothing
};

}  // namespace

struct gmcp_fem {
  hipStream_t stream;
  int64_t V, n_tet, nnzb, n_slices;
  double mu, lambda, rho, dt;
  FemDev d;
  double *host;                 // pinned: residuals the device reports (two rr, bb pairs)
  hipEvent_t ev[2];             // recorded after each report
  std::vector<uint8_t> hfixed;  // host copy of the Dirichlet component masks
};

namespace {

__device__ inline void shape_grads(const double *X, const int32_t *tet, double g[4][3], double *vol) {
  double a[3], b[3], c[3];
  const double *x0 = X + 3 * (int64_t)tet[0];
  for (int d = 0; d < 3; ++d) {
    a[d] = X[3 * (int64_t)tet[1] + d] - x0[d];
    b[d] = X[3 * (int64_t)tet[2] + d] - x0[d];
    c[d] = X[3 * (int64_t)tet[3] + d] - x0[d];
  }
  // Dm = [a b c] (columns); rows of Dm^{-1} are the gradients of N_1..N_3
  double det = a[0] * (b[1] * c[2] - b[2] * c[1]) - b[0] * (a[1] * c[2] - a[2] * c[1]) +
               c[0] * (a[1] * b[2] - a[2] * b[1]);
  double id = 1.0 / det;
  // inverse rows = (b x c, c x a, a x b) / det
  double r1[3] = {b[1] * c[2] - b[2] * c[1], b[2] * c[0] - b[0] * c[2], b[0] * c[1] - b[1] * c[0]};
  double r2[3] = {c[1] * a[2] - c[2] * a[1], c[2] * a[0] - c[0] * a[2], c[0] * a[1] - c[1] * a[0]};
  double r3[3] = {a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]};
  for (int d = 0; d < 3; ++d) {
    g[1][d] = r1[d] * id;
    g[2][d] = r2[d] * id;
    g[3][d] = r3[d] * id;
    g[0][d] = -(g[1][d] + g[2][d] + g[3][d]);
  }
  *vol = fabs(det) / 6.0;
}

// where value z of K's block bk is kept: entry bk - row_ptr[row] of the row's slice
__device__ inline int64_t sell_at(const int32_t *s_off, const int32_t *krp, int64_t row, int64_t bk) {
  return ((int64_t)s_off[row / kSlice] + (bk - krp[row])) * 9 * kSlice + row % kSlice;
}

__global__ void k_kvals(const double *X, const int32_t *tets, const int32_t *c_off, const int32_t *c_list,
                        int64_t nnzb, double mu, double lambda, const int32_t *k_row, const int32_t *krp,
                        const int32_t *s_off, double *s_val) {
  int64_t bk = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (bk >= nnzb) return;
  double K[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  for (int c = c_off[bk]; c < c_off[bk + 1]; ++c) {
    int code = c_list[c];
    int t = code >> 4, a = (code >> 2) & 3, b = code & 3;
    double g[4][3], vol;
    shape_grads(X, tets + 4 * (int64_t)t, g, &vol);
    double dab = g[a][0] * g[b][0] + g[a][1] * g[b][1] + g[a][2] * g[b][2];
    for (int i = 0; i < 3; ++i)
      for (int k = 0; k < 3; ++k)
        K[3 * i + k] += vol * (mu * (i == k ? dab : 0.0) + mu * g[b][i] * g[a][k] + lambda * g[a][i] * g[b][k]);
  }
  const int64_t at = sell_at(s_off, krp, k_row[bk], bk);
  for (int z = 0; z < 9; ++z) s_val[at + z * kSlice] = K[z];
}

// K's blocks in row order (gmcp_fem_stiffness)
__global__ void k_export(const int32_t *k_row, const int32_t *krp, const int32_t *s_off, const double *s_val,
                         int64_t nnzb, double *val) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= 9 * nnzb) return;
  const int64_t bk = i / 9;
  val[i] = s_val[sell_at(s_off, krp, k_row[bk], bk) + (i - 9 * bk) * kSlice];
}

// component d of vertex c, 0 when that component is held (Dirichlet
// columns removed)
__device__ inline void free_part(const double *x, const uint8_t *fixed, int64_t c, double v[3]) {
  const int m = fixed[c];
  for (int d = 0; d < 3; ++d) v[d] = (m >> d) & 1 ? 0.0 : x[3 * c + d];
}

// s = K v + H v of row `slice * 64 + lane` for NV vectors at once, v(c) from
// load(c, v): the block's four waves take every fourth block of the row and
// wave 0 adds their sums in wave order (its s is the row's; the other waves'
// are partial).  Every thread of the block calls it.
template <int NV, typename Load>
__device__ inline void row_products(const Sell &K, const int32_t *__restrict__ hrp, const int32_t *__restrict__ hcol,
                                    const double *__restrict__ hval, int64_t slice, int64_t V, Load load,
                                    double s[NV][3]) {
  __shared__ double red[kSliceWaves - 1][3 * NV][kSlice];
  const int w = threadIdx.x / kSlice, lane = threadIdx.x % kSlice;
  const int64_t i = slice * kSlice + lane;
  int h0 = 0, h1 = 0;
  if (hrp && i < V) {
    h0 = hrp[i] + w;
    h1 = hrp[i + 1];
  }
  for (int n = 0; n < NV; ++n) s[n][0] = s[n][1] = s[n][2] = 0.0;
  const int e1 = K.off[slice + 1];
  // two entries at a time, so that both columns' vectors are in flight
  // beside the values
  for (int e = K.off[slice] + w; e < e1; e += 2 * kSliceWaves) {
    const bool two = e + kSliceWaves < e1;
    int32_t c[2];
    double B[2][9], v[2][NV][3];
    c[0] = K.col[(int64_t)e * kSlice + lane];
    c[1] = two ? K.col[(int64_t)(e + kSliceWaves) * kSlice + lane] : -1;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      for (int n = 0; n < NV; ++n) v[k][n][0] = v[k][n][1] = v[k][n][2] = 0.0;
#pragma unroll
      for (int z = 0; z < 9; ++z)
        B[k][z] = c[k] < 0 ? 0.0 : K.val[((int64_t)(e + k * kSliceWaves) * 9 + z) * kSlice + lane];
    }
#pragma unroll
    for (int k = 0; k < 2; ++k)
      if (c[k] >= 0) load(c[k], v[k]);
#pragma unroll
    for (int k = 0; k < 2; ++k)
      for (int n = 0; n < NV; ++n)
        for (int r = 0; r < 3; ++r)
          s[n][r] += B[k][3 * r] * v[k][n][0] + B[k][3 * r + 1] * v[k][n][1] + B[k][3 * r + 2] * v[k][n][2];
  }
  for (int j = h0; j < h1; j += kSliceWaves) {
    double v[NV][3];
    load(hcol[j], v);
    const double *B = hval + 9 * (int64_t)j;
    for (int n = 0; n < NV; ++n)
      for (int r = 0; r < 3; ++r) s[n][r] += B[3 * r] * v[n][0] + B[3 * r + 1] * v[n][1] + B[3 * r + 2] * v[n][2];
  }
  if (w > 0)
    for (int n = 0; n < NV; ++n)
      for (int r = 0; r < 3; ++r) red[w - 1][3 * n + r][lane] = s[n][r];
  __syncthreads();
  if (w == 0)
    for (int k = 0; k < kSliceWaves - 1; ++k)
      for (int n = 0; n < NV; ++n)
        for (int r = 0; r < 3; ++r) s[n][r] += red[k][3 * n + r][lane];
}

// sum over a wave (fixed butterfly); every lane gets it
__device__ inline double wave_sum(double v) {
  for (int o = kSlice / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kSlice);
  return v;
}

// sum of n partials by one wave, in a fixed order (lane l adds l, l + 64,
// ...), ten loads in flight
__device__ inline double sum_partials(const double *__restrict__ part, int n) {
  const int lane = threadIdx.x % kSlice;
  double v = 0.0;
  for (int j0 = lane; j0 < n; j0 += 10 * kSlice) {
    double t[10];
#pragma unroll
    for (int k = 0; k < 10; ++k) t[k] = j0 + k * kSlice < n ? part[j0 + k * kSlice] : 0.0;
#pragma unroll
    for (int k = 0; k < 10; ++k) v += t[k];
  }
  return wave_sum(v);
}

// sum over a block of kT threads (fixed order), valid in thread 0
__device__ inline double block_sum(double v) {
  __shared__ double ws[kT / kSlice];
  v = wave_sum(v);
  __syncthreads();  // an earlier sum's reads are done
  if (threadIdx.x % kSlice == 0) ws[threadIdx.x / kSlice] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int k = 0; k < kT / kSlice; ++k) t += ws[k];
  return t;
}

// y = (M/dt^2) x + K x + H x (H optional) over the free components; 0 in
// the held ones
__global__ __launch_bounds__(kSlice *kSliceWaves) void k_apply(Sell K, const int32_t *__restrict__ hrp,
                                                               const int32_t *__restrict__ hcol,
                                                               const double *__restrict__ hval,
                                                               const double *__restrict__ mass,
                                                               const uint8_t *__restrict__ fixed, double inv_dt2,
                                                               const double *__restrict__ x, double *__restrict__ y,
                                                               int64_t V) {
  const int64_t i = (int64_t)blockIdx.x * kSlice + threadIdx.x;
  double s[1][3];
  row_products<1>(K, hrp, hcol, hval, blockIdx.x, V, [&](int64_t c, double (*v)[3]) { free_part(x, fixed, c, v[0]); },
                  s);
  if (threadIdx.x >= kSlice || i >= V) return;
  const int mi = fixed[i];
  double v[3];
  free_part(x, fixed, i, v);
  for (int d = 0; d < 3; ++d) y[3 * i + d] = (mi >> d) & 1 ? 0.0 : mass[i] * inv_dt2 * v[d] + s[0][d];
}

__device__ inline bool inv3(const double *A, double *B) {
  double c00 = A[4] * A[8] - A[5] * A[7], c01 = A[5] * A[6] - A[3] * A[8], c02 = A[3] * A[7] - A[4] * A[6];
  double det = A[0] * c00 + A[1] * c01 + A[2] * c02;
  if (!(fabs(det) > 0.0)) return false;
  double id = 1.0 / det;
  B[0] = c00 * id;
  B[1] = (A[2] * A[7] - A[1] * A[8]) * id;
  B[2] = (A[1] * A[5] - A[2] * A[4]) * id;
  B[3] = c01 * id;
  B[4] = (A[0] * A[8] - A[2] * A[6]) * id;
  B[5] = (A[2] * A[3] - A[0] * A[5]) * id;
  B[6] = c02 * id;
  B[7] = (A[1] * A[6] - A[0] * A[7]) * id;
  B[8] = (A[0] * A[4] - A[1] * A[3]) * id;
  return true;
}

// ---------------------------------------------------------------- CG
// Device scalars: scal[0], scal[1] = r.z of the even and odd iterations,
// scal[2] = b.b, scal[3] = r.r at the last check.
//
// An iteration is two launches.  The dot products' block partials are summed
// (in a fixed order) by every block of the launch that needs them, so no
// launch of its own finishes them, and the new search direction is formed
// where it is read.  Seven launches per iteration (product, two partial and
// two final dots, update, preconditioner, direction, scalar) took 48 us at
// 38025 vertices, 22.8 us of it the product.

// block-Jacobi inverse, x = 0, r = b over the free components, z = P r and
// the partials of r.z and b.b
__global__ __launch_bounds__(kT) void k_cg_init(Sell K, const int32_t *__restrict__ s_off,
                                                const int32_t *__restrict__ krp,
                                                const int32_t *__restrict__ k_diag, const int32_t *__restrict__ hrp,
                                                const int32_t *__restrict__ hcol, const double *__restrict__ hval,
                                                const double *__restrict__ mass, const uint8_t *__restrict__ fixed,
                                                double inv_dt2, const double *__restrict__ rhs,
                                                double *__restrict__ Pinv, double *__restrict__ x,
                                                double *__restrict__ rv, double *__restrict__ zv,
                                                double *__restrict__ part_rz, double *__restrict__ part_rr,
                                                int32_t *done, int64_t V) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i == 0) *done = 0;
  double rz = 0.0, rr = 0.0;
  if (i < V) {
    double D[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (int d = 0; d < 3; ++d) D[4 * d] = mass[i] * inv_dt2;
    const int32_t dg = k_diag[i];
    if (dg >= 0) {
      const double *B = K.val + sell_at(s_off, krp, i, dg);
      for (int z = 0; z < 9; ++z) D[z] += B[z * kSlice];
    }
    if (hrp)
      for (int j = hrp[i]; j < hrp[i + 1]; ++j)
        if (hcol[j] == i)
          for (int z = 0; z < 9; ++z) D[z] += hval[9 * (int64_t)j + z];
    // held components: identity rows/columns for the inverse, zeroed after
    const int m = fixed[i];
    for (int d = 0; d < 3; ++d)
      if ((m >> d) & 1)
        for (int k = 0; k < 3; ++k) D[3 * d + k] = D[3 * k + d] = (k == d) ? 1.0 : 0.0;
    double P[9];
    if (m == 7 || !inv3(D, P))
      for (int z = 0; z < 9; ++z) P[z] = 0.0;
    for (int d = 0; d < 3; ++d)
      if ((m >> d) & 1)
        for (int k = 0; k < 3; ++k) P[3 * d + k] = P[3 * k + d] = 0.0;
    for (int z = 0; z < 9; ++z) Pinv[9 * i + z] = P[z];
    double b[3];
    free_part(rhs, fixed, i, b);
    for (int d = 0; d < 3; ++d) {
      const double z = P[3 * d] * b[0] + P[3 * d + 1] * b[1] + P[3 * d + 2] * b[2];
      x[3 * i + d] = 0.0;
      rv[3 * i + d] = b[d];
      zv[3 * i + d] = z;
      rz += b[d] * z;
      rr += b[d] * b[d];
    }
  }
  const double srz = block_sum(rz), srr = block_sum(rr);
  if (threadIdx.x == 0) {
    part_rz[blockIdx.x] = srz;
    part_rr[blockIdx.x] = srr;
  }
}

// p = z + beta p_old (beta = rz / rz_old, 0 in the first iteration), q = A p
// and the partials of p.q.  p is 0 in held components (z is, by Pinv), so
// the columns need no mask.  The row sums A z and A p_old run side by side
// and meet beta at the end, so the sum of r.z's partials and the done flag
// are waited for after the matrix has been read, not before.
__global__ __launch_bounds__(kSlice *kSliceWaves) void k_cg_apply(
    Sell K, const int32_t *__restrict__ hrp, const int32_t *__restrict__ hcol, const double *__restrict__ hval,
    const double *__restrict__ mass, const uint8_t *__restrict__ fixed, double inv_dt2,
    const double *__restrict__ z, const double *__restrict__ p_old, double *__restrict__ p, double *__restrict__ q,
    const double *__restrict__ part_rz, int n_rz, double *__restrict__ scal, int parity, int first,
    double *__restrict__ part_pq, const int32_t *__restrict__ done, int64_t V) {
  double s[2][3];
  row_products<2>(
      K, hrp, hcol, hval, blockIdx.x, V,
      [&](int64_t c, double (*v)[3]) {
        for (int d = 0; d < 3; ++d) {
          v[0][d] = z[3 * c + d];
          v[1][d] = first ? 0.0 : p_old[3 * c + d];
        }
      },
      s);
  if (threadIdx.x >= kSlice || *done) return;
  const double rz = sum_partials(part_rz, n_rz), rz_old = first ? 0.0 : scal[parity ^ 1];
  const double beta = rz_old != 0.0 ? rz / rz_old : 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) scal[parity] = rz;
  const int64_t i = (int64_t)blockIdx.x * kSlice + threadIdx.x;
  double pq = 0.0;
  if (i < V) {
    const int mi = fixed[i];
    for (int d = 0; d < 3; ++d) {
      const double v = first ? z[3 * i + d] : z[3 * i + d] + beta * p_old[3 * i + d];
      const double qd = (mi >> d) & 1 ? 0.0 : mass[i] * inv_dt2 * v + (s[0][d] + beta * s[1][d]);
      p[3 * i + d] = v;
      q[3 * i + d] = qd;
      pq += v * qd;
    }
  }
  pq = wave_sum(pq);
  if (threadIdx.x == 0) part_pq[blockIdx.x] = pq;
}

// x += alpha p, r -= alpha q (alpha = rz / p.q), z = P r and the partials of
// r.z and r.r
__global__ __launch_bounds__(kT) void k_cg_update(const double *__restrict__ Pinv, const double *__restrict__ p,
                                                  const double *__restrict__ q, double *__restrict__ x,
                                                  double *__restrict__ rv, double *__restrict__ zv,
                                                  const double *__restrict__ part_pq, int n_pq,
                                                  const double *__restrict__ scal, int parity,
                                                  double *__restrict__ part_rz, double *__restrict__ part_rr,
                                                  const int32_t *__restrict__ done, int64_t V) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  double rz = 0.0, rr = 0.0;
  // the vertex's values first: they are in flight while the partials are summed
  double P[9], xi[3], r[3], pi[3], qi[3];
  if (i < V) {
    for (int k = 0; k < 9; ++k) P[k] = Pinv[9 * i + k];
    for (int d = 0; d < 3; ++d) {
      xi[d] = x[3 * i + d];
      r[d] = rv[3 * i + d];
      pi[d] = p[3 * i + d];
      qi[d] = q[3 * i + d];
    }
  }
  const double pq = sum_partials(part_pq, n_pq);
  const double alpha = pq != 0.0 ? scal[parity] / pq : 0.0;
  if (*done) return;
  if (i < V) {
    for (int d = 0; d < 3; ++d) {
      x[3 * i + d] = xi[d] + alpha * pi[d];
      r[d] -= alpha * qi[d];
      rv[3 * i + d] = r[d];
      rr += r[d] * r[d];
    }
    for (int d = 0; d < 3; ++d) {
      const double z = P[3 * d] * r[0] + P[3 * d + 1] * r[1] + P[3 * d + 2] * r[2];
      zv[3 * i + d] = z;
      rz += r[d] * z;
    }
  }
  const double srz = block_sum(rz), srr = block_sum(rr);
  if (threadIdx.x == 0) {
    part_rz[blockIdx.x] = srz;
    part_rr[blockIdx.x] = srr;
  }
}

// r.r against the tolerance (start: it is b.b), reported to the host; ends
// the CG on the device, so that launches already queued leave x alone
__global__ __launch_bounds__(kSlice) void k_cg_check(const double *__restrict__ part_rr, int n, double *scal,
                                                     int start, double rtol2, int32_t *done, double *host) {
  if (*done) return;
  const double rr = sum_partials(part_rr, n);
  if (threadIdx.x != 0) return;
  if (start) scal[2] = rr;
  const double bb = start ? rr : scal[2];
  scal[3] = rr;
  if (start ? !(bb > 0.0) : rr <= rtol2 * bb) *done = 1;
  host[0] = rr;
  host[1] = bb;
  __threadfence_system();
}

// elastic + inertial energy terms per vertex and gradient:
//   g_i = m_i (x_i - xt_i)/dt^2 + (K (x - X))_i ; 0 in held components
//   e_i = 1/2 m_i |x_i - xt_i|^2 / dt^2 + 1/2 u_i . (K u)_i
// with the energy's partial per slice
__global__ __launch_bounds__(kSlice *kSliceWaves) void k_fem_grad(Sell K, const double *__restrict__ mass,
                                                                  const uint8_t *__restrict__ fixed, double inv_dt2,
                                                                  const double *__restrict__ X,
                                                                  const double *__restrict__ x,
                                                                  const double *__restrict__ xt, double *g,
                                                                  double *__restrict__ part, int64_t V) {
  double ku[1][3];
  row_products<1>(
      K, nullptr, nullptr, nullptr, blockIdx.x, V,
      [&](int64_t c, double (*u)[3]) {
        for (int d = 0; d < 3; ++d) u[0][d] = x[3 * c + d] - X[3 * c + d];
      },
      ku);
  if (threadIdx.x >= kSlice) return;
  const int64_t i = (int64_t)blockIdx.x * kSlice + threadIdx.x;
  double ei = 0.0;
  if (i < V)
    for (int d = 0; d < 3; ++d) {
      double dv = x[3 * i + d] - xt[3 * i + d];
      double ui = x[3 * i + d] - X[3 * i + d];
      ei += 0.5 * mass[i] * inv_dt2 * dv * dv + 0.5 * ui * ku[0][d];
      if (g) g[3 * i + d] = (fixed[i] >> d) & 1 ? 0.0 : mass[i] * inv_dt2 * dv + ku[0][d];
    }
  ei = wave_sum(ei);
  if (threadIdx.x == 0) part[blockIdx.x] = ei;
}

__global__ __launch_bounds__(kT) void k_sum(const double *__restrict__ part, int64_t n, double *out) {
  double v = 0.0;
  for (int64_t j = threadIdx.x; j < n; j += kT) v += part[j];
  v = block_sum(v);
  if (threadIdx.x == 0) *out = v;
}

inline unsigned nb(int64_t n) { return (unsigned)((n + kT - 1) / kT); }

struct FemPlan {
  size_t off = 0;
  char *base = nullptr;
  template <typename T>
  T *take(int64_t n) {
    off = (off + 255) & ~size_t(255);
    T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
    off += sizeof(T) * (size_t)(n > 0 ? n : 1);
    return p;
  }
};

struct FemTopo {
  std::vector<int32_t> rp, col, coff, clist;
  std::vector<int32_t> row, diag, soff;  // row of each block, diagonal block of each row, slices' first entries
};

void fem_topology(const int32_t *tets, int64_t n_tet, int64_t V, FemTopo &t) {
  std::vector<std::map<int32_t, std::vector<int32_t>>> rows(V);
  for (int64_t e = 0; e < n_tet; ++e)
    for (int a = 0; a < 4; ++a)
      for (int b = 0; b < 4; ++b) rows[tets[4 * e + a]][tets[4 * e + b]].push_back((int32_t)(e * 16 + a * 4 + b));
  t.rp.assign(V + 1, 0);
  for (int64_t i = 0; i < V; ++i) t.rp[i + 1] = t.rp[i] + (int32_t)rows[i].size();
  t.col.clear();
  t.coff.assign(1, 0);
  t.clist.clear();
  for (int64_t i = 0; i < V; ++i)
    for (auto &kv : rows[i]) {
      t.col.push_back(kv.first);
      for (int32_t c : kv.second) t.clist.push_back(c);
      t.coff.push_back((int32_t)t.clist.size());
    }
  t.row.resize(t.col.size());
  t.diag.assign(V, -1);
  t.soff.assign((V + kSlice - 1) / kSlice + 1, 0);
  for (int64_t i = 0; i < V; ++i) {
    int32_t &width = t.soff[i / kSlice + 1];  // the slice's longest row
    width = std::max(width, t.rp[i + 1] - t.rp[i]);
    for (int32_t k = t.rp[i]; k < t.rp[i + 1]; ++k) {
      t.row[k] = (int32_t)i;
      if (t.col[k] == i) t.diag[i] = k;
    }
  }
  for (size_t k = 1; k < t.soff.size(); ++k) t.soff[k] += t.soff[k - 1];
}

size_t fem_plan(int64_t V, int64_t n_tet, const FemTopo &topo, char *base, FemDev *d) {
  FemPlan p;
  p.base = base;
  FemDev t{};
  const int64_t n = 3 * V, nnzb = (int64_t)topo.col.size(), entries = topo.soff.back();
  t.k_row_ptr = p.take<int32_t>(V + 1);
  t.k_col = p.take<int32_t>(nnzb);
  t.k_row = p.take<int32_t>(nnzb);
  t.s_off = p.take<int32_t>((int64_t)topo.soff.size());
  t.s_col = p.take<int32_t>(entries * kSlice);
  t.s_val = p.take<double>(9 * entries * kSlice);
  t.k_diag = p.take<int32_t>(V);
  t.c_off = p.take<int32_t>(nnzb + 1);
  t.c_list = p.take<int32_t>((int64_t)topo.clist.size());
  t.mass = p.take<double>(V);
  t.fixed = p.take<uint8_t>(V);
  t.X = p.take<double>(3 * V);
  t.tets = p.take<int32_t>(4 * n_tet);
  t.Pinv = p.take<double>(9 * V);
  t.r = p.take<double>(n);
  t.z = p.take<double>(n);
  t.q = p.take<double>(n);
  for (int k = 0; k < 2; ++k) t.p[k] = p.take<double>(n);
  t.part_pq = p.take<double>((V + kSlice - 1) / kSlice);
  t.part_rz = p.take<double>((V + kT - 1) / kT);
  t.part_rr = p.take<double>((V + kT - 1) / kT);
  t.scal = p.take<double>(16);
  t.done = p.take<int32_t>(1);
  if (d) *d = t;
  return p.off + 256;
}

inline Sell sell(const FemDev &d) { return Sell{d.s_off, d.s_col, d.s_val}; }

}  // namespace

extern "C" {

size_t gmcp_fem_workspace_size(const int32_t *tets, int64_t n_tet, int64_t n_vert) {
  if (!tets || n_tet <= 0 || n_vert <= 0) return 0;
  for (int64_t i = 0; i < 4 * n_tet; ++i)
    if (tets[i] < 0 || tets[i] >= n_vert) return 0;
  FemTopo t;
  fem_topology(tets, n_tet, n_vert, t);
  return fem_plan(n_vert, n_tet, t, nullptr, nullptr);
}

int gmcp_fem_create(gmcp_fem **out, const int32_t *tets, int64_t n_tet, int64_t n_vert, const double *X_rest,
                    double young, double poisson, double density, double dt, const int32_t *fixed,
                    int64_t n_fixed, void *workspace, size_t bytes, void *stream) {
  if (!out || !X_rest || !(young > 0) || !(poisson > -1 && poisson < 0.5) || !(density > 0) || !(dt > 0))
    return GMCP_E_ARG;
  *out = nullptr;
  size_t need = gmcp_fem_workspace_size(tets, n_tet, n_vert);
  if (need == 0 || bytes < need || !workspace || (reinterpret_cast<uintptr_t>(workspace) & 255)) return GMCP_E_ARG;
  for (int64_t i = 0; i < n_fixed; ++i)
    if (fixed[i] < 0 || fixed[i] >= n_vert) return GMCP_E_ARG;
  FemTopo t;
  fem_topology(tets, n_tet, n_vert, t);
  gmcp_fem *f = new (std::nothrow) gmcp_fem();
  if (!f) return GMCP_E_ARG;
  f->stream = (hipStream_t)stream;
  f->V = n_vert;
  f->n_tet = n_tet;
  f->nnzb = (int64_t)t.col.size();
  f->mu = young / (2.0 * (1.0 + poisson));
  f->lambda = young * poisson / ((1.0 + poisson) * (1.0 - 2.0 * poisson));
  f->rho = density;
  f->dt = dt;
  f->n_slices = (int64_t)t.soff.size() - 1;
  f->host = nullptr;
  f->ev[0] = f->ev[1] = nullptr;
  fem_plan(n_vert, n_tet, t, (char *)workspace, &f->d);
  // the slices' columns; rows shorter than their slice end in -1
  std::vector<int32_t> scol((size_t)t.soff.back() * kSlice, -1);
  for (size_t k = 0; k < t.col.size(); ++k) {
    const int32_t i = t.row[k];
    scol[((size_t)t.soff[i / kSlice] + (k - t.rp[i])) * kSlice + i % kSlice] = t.col[k];
  }
  // lumped mass: rho vol / 4 per tet vertex
  std::vector<double> mass(n_vert, 0.0);
  for (int64_t e = 0; e < n_tet; ++e) {
    const double *x0 = X_rest + 3 * (int64_t)tets[4 * e];
    double a[3], b[3], c[3];
    for (int d = 0; d < 3; ++d) {
      a[d] = X_rest[3 * (int64_t)tets[4 * e + 1] + d] - x0[d];
      b[d] = X_rest[3 * (int64_t)tets[4 * e + 2] + d] - x0[d];
      c[d] = X_rest[3 * (int64_t)tets[4 * e + 3] + d] - x0[d];
    }
    double det = a[0] * (b[1] * c[2] - b[2] * c[1]) - b[0] * (a[1] * c[2] - a[2] * c[1]) +
                 c[0] * (a[1] * b[2] - a[2] * b[1]);
    for (int k = 0; k < 4; ++k) mass[tets[4 * e + k]] += density * fabs(det) / 24.0;
  }
  std::vector<uint8_t> fx(n_vert, 0);
  for (int64_t i = 0; i < n_fixed; ++i) fx[fixed[i]] = 7;
  hipError_t e = hipSuccess;
  auto up = [&](void *dst, const void *src, size_t n) {
    if (e == hipSuccess && n) e = hipMemcpy(dst, src, n, hipMemcpyHostToDevice);
  };
  up(f->d.k_row_ptr, t.rp.data(), sizeof(int32_t) * t.rp.size());
  up(f->d.k_col, t.col.data(), sizeof(int32_t) * t.col.size());
  up(f->d.k_row, t.row.data(), sizeof(int32_t) * t.row.size());
  up(f->d.s_off, t.soff.data(), sizeof(int32_t) * t.soff.size());
  up(f->d.s_col, scol.data(), sizeof(int32_t) * scol.size());
  up(f->d.k_diag, t.diag.data(), sizeof(int32_t) * t.diag.size());
  up(f->d.c_off, t.coff.data(), sizeof(int32_t) * t.coff.size());
  up(f->d.c_list, t.clist.data(), sizeof(int32_t) * t.clist.size());
  up(f->d.mass, mass.data(), sizeof(double) * n_vert);
  up(f->d.fixed, fx.data(), n_vert);
  f->hfixed = fx;
  up(f->d.X, X_rest, sizeof(double) * 3 * n_vert);
  up(f->d.tets, tets, sizeof(int32_t) * 4 * n_tet);
  if (e == hipSuccess) e = hipHostMalloc((void **)&f->host, 4 * sizeof(double), hipHostMallocCoherent);
  for (int k = 0; k < 2; ++k)
    if (e == hipSuccess) e = hipEventCreateWithFlags(&f->ev[k], hipEventDisableTiming);
  if (e != hipSuccess) {
    gmcp_fem_destroy(f);
    return GMCP_E_HIP;
  }
  hipLaunchKernelGGL(k_kvals, dim3(nb(f->nnzb)), dim3(kT), 0, f->stream, f->d.X, f->d.tets, f->d.c_off, f->d.c_list,
                     f->nnzb, f->mu, f->lambda, f->d.k_row, f->d.k_row_ptr, f->d.s_off, f->d.s_val);
  if (hipGetLastError() != hipSuccess || hipStreamSynchronize(f->stream) != hipSuccess) {
    gmcp_fem_destroy(f);
    return GMCP_E_HIP;
  }
  *out = f;
  return GMCP_OK;
}

void gmcp_fem_destroy(gmcp_fem *f) {
  if (!f) return;
  for (int k = 0; k < 2; ++k)
    if (f->ev[k]) (void)hipEventDestroy(f->ev[k]);
  if (f->host) (void)hipHostFree(f->host);
  delete f;
}

int gmcp_fem_constrain(gmcp_fem *f, const int32_t *verts, int64_t n, int mask) {
  if (!f || n < 0 || (n > 0 && !verts) || mask < 1 || mask > 7) return GMCP_E_ARG;
  for (int64_t i = 0; i < n; ++i)
    if (verts[i] < 0 || verts[i] >= f->V) return GMCP_E_ARG;
  for (int64_t i = 0; i < n; ++i) f->hfixed[verts[i]] |= (uint8_t)mask;
  if (hipStreamSynchronize(f->stream) != hipSuccess ||
      hipMemcpy(f->d.fixed, f->hfixed.data(), (size_t)f->V, hipMemcpyHostToDevice) != hipSuccess)
    return GMCP_E_HIP;
  return GMCP_OK;
}

int gmcp_fem_set_stream(gmcp_fem *f, void *stream) {
  if (!f) return GMCP_E_ARG;
  f->stream = (hipStream_t)stream;
  return GMCP_OK;
}

int64_t gmcp_fem_nnzb(const gmcp_fem *f) { return f ? f->nnzb : -1; }

int gmcp_fem_stiffness(gmcp_fem *f, int32_t *row_ptr, int32_t *col, double *val) {
  if (!f || !row_ptr || !col || !val) return GMCP_E_ARG;
  hipError_t e = hipMemcpyAsync(row_ptr, f->d.k_row_ptr, sizeof(int32_t) * (f->V + 1), hipMemcpyDeviceToDevice, f->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(col, f->d.k_col, sizeof(int32_t) * f->nnzb, hipMemcpyDeviceToDevice, f->stream);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_export, dim3(nb(9 * f->nnzb)), dim3(kT), 0, f->stream, f->d.k_row, f->d.k_row_ptr, f->d.s_off,
                       f->d.s_val, f->nnzb, val);
    e = hipGetLastError();
  }
  return e == hipSuccess ? GMCP_OK : GMCP_E_HIP;
}

int gmcp_fem_energy(gmcp_fem *f, const double *x, const double *x_tilde, double *energy, double *grad) {
  if (!f || !x || !x_tilde || !energy) return GMCP_E_ARG;
  double inv_dt2 = 1.0 / (f->dt * f->dt);
  hipLaunchKernelGGL(k_fem_grad, dim3((unsigned)f->n_slices), dim3(kSlice * kSliceWaves), 0, f->stream, sell(f->d),
                     f->d.mass, f->d.fixed, inv_dt2, f->d.X, x, x_tilde, grad, f->d.part_pq, f->V);
  hipLaunchKernelGGL(k_sum, dim3(1), dim3(kT), 0, f->stream, f->d.part_pq, f->n_slices, energy);
  return hipGetLastError() == hipSuccess ? GMCP_OK : GMCP_E_HIP;
}

int gmcp_fem_solve(gmcp_fem *f, const int32_t *h_row_ptr, const int32_t *h_col, const double *h_val,
                   const double *rhs, double *x, double rtol, int max_iter, int *iters, double *rel_res) {
  if (!f || !rhs || !x || max_iter <= 0 || !(rtol > 0)) return GMCP_E_ARG;
  if ((h_row_ptr != nullptr) != (h_col != nullptr) || (h_col != nullptr) != (h_val != nullptr)) return GMCP_E_ARG;
  hipStream_t s = f->stream;
  const int64_t V = f->V;
  const double inv_dt2 = 1.0 / (f->dt * f->dt);
  FemDev &d = f->d;
  const int n_rz = (int)nb(V), n_pq = (int)f->n_slices;
  const double rtol2 = rtol * rtol;
  hipLaunchKernelGGL(k_cg_init, dim3(nb(V)), dim3(kT), 0, s, sell(d), d.s_off, d.k_row_ptr, d.k_diag, h_row_ptr,
                     h_col, h_val, d.mass, d.fixed, inv_dt2, rhs, d.Pinv, x, d.r, d.z, d.part_rz, d.part_rr, d.done,
                     V);
  hipLaunchKernelGGL(k_cg_check, dim3(1), dim3(kSlice), 0, s, d.part_rr, n_rz, d.scal, 1, rtol2, d.done, f->host);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipEventRecord(f->ev[0], s);
  // Eight iterations between checks of the residual.  The host reads check
  // c while the iterations after it run; those queued past the end do
  // nothing (the device holds the decision), so x is that of the check.
  int it = 0, queued = 0, end = 0;
  int upto[2] = {0, 0};  // iterations done at the check in each slot
  double rr = 0.0, bb = 0.0;
  for (int c = 0; e == hipSuccess; ++c) {
    if (queued < max_iter) {
      end = std::min(max_iter, queued + 8 - queued % 8);
      for (; queued < end; ++queued) {
        const int par = queued & 1;
        hipLaunchKernelGGL(k_cg_apply, dim3(n_pq), dim3(kSlice * kSliceWaves), 0, s, sell(d), h_row_ptr, h_col, h_val,
                           d.mass, d.fixed, inv_dt2, d.z, d.p[par ^ 1], d.p[par], d.q, d.part_rz, n_rz, d.scal, par,
                           queued == 0 ? 1 : 0, d.part_pq, d.done, V);
        hipLaunchKernelGGL(k_cg_update, dim3(n_rz), dim3(kT), 0, s, d.Pinv, d.p[par], d.q, x, d.r, d.z, d.part_pq,
                           n_pq, d.scal, par, d.part_rz, d.part_rr, d.done, V);
      }
      const int slot = (c + 1) & 1;
      upto[slot] = queued;
      hipLaunchKernelGGL(k_cg_check, dim3(1), dim3(kSlice), 0, s, d.part_rr, n_rz, d.scal, 0, rtol2, d.done,
                         f->host + 2 * slot);
      e = hipGetLastError();
      if (e == hipSuccess) e = hipEventRecord(f->ev[slot], s);
      if (e != hipSuccess) break;
    }
    if ((e = hipEventSynchronize(f->ev[c & 1])) != hipSuccess) break;
    const volatile double *said = f->host + 2 * (c & 1);
    rr = said[0];
    bb = said[1];
    it = upto[c & 1];
    if (c == 0 ? !(bb > 0.0) : (!(rr == rr) || rr <= rtol2 * bb || it >= max_iter)) break;
  }
  // nothing is left in flight when the call returns
  if (e != hipSuccess || hipStreamSynchronize(s) != hipSuccess) return GMCP_E_HIP;
  if (bb > 0.0 && !(rr == rr)) return GMCP_E_NONFINITE;
  if (iters) *iters = it;
  if (rel_res) *rel_res = bb > 0.0 ? sqrt(rr / bb) : 0.0;
  return hipGetLastError() == hipSuccess ? GMCP_OK : GMCP_E_HIP;
}

// y = A x (for checks): A = M/dt^2 + K + H, fixed rows 0
int gmcp_fem_apply(gmcp_fem *f, const int32_t *h_row_ptr, const int32_t *h_col, const double *h_val, const double *x,
                   double *y) {
  if (!f || !x || !y) return GMCP_E_ARG;
  hipLaunchKernelGGL(k_apply, dim3((unsigned)f->n_slices), dim3(kSlice * kSliceWaves), 0, f->stream, sell(f->d),
                     h_row_ptr, h_col, h_val, f->d.mass, f->d.fixed, 1.0 / (f->dt * f->dt), x, y, f->V);
  return hipGetLastError() == hipSuccess ? GMCP_OK : GMCP_E_HIP;
}

}  // extern "C"
