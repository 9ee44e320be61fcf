// Exact coarse solve F_c^{-1} by block elimination in time (the coarse
// operator is block tridiagonal in time, Section 3.2; block k = the 3 N_c
// unknowns of coarse level k):
//   S_0 = D_0,  S_k = D_k - L_k S_{k-1}^{-1} U_{k-1},
//   forward   y_0 = S_0^{-1} r_0,  y_k = S_k^{-1} (r_k - L_k y_{k-1}),
//   backward  x_M = y_M,           x_k = y_k - E_k x_{k+1},  E_k = S_k^{-1} U_k.
// D_k, L_k, U_k are the stencil blocks of the coarse operator (its 27 spatial
// neighbours at time offsets 0, -1, +1).  The setup forms every S_k densely
// and inverts it explicitly (blocked Gauss-Jordan elimination with partial
// pivoting, the trailing updates as tiled FP64 GEMMs), so one application is
// two sweeps of dense block products streamed from HBM: matrix-vector
// products (solve) or matrix-core products for up to 16 vectors per pass
// (solve_multi).
//
// Dense matrices are stored column-major (entry (r, c) at c * nb + r during
// the setup; the kept S_k^{-1} and E_k at c * ld + r, ld = nb rounded up to
// 64).  The Gauss-Jordan kernels work on rows of the buffer, i.e. on the
// transpose; the inverse of the transpose read column-major is the inverse
// itself.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <vector>

#include "coarse_lu.hpp"
#include "stencil.hpp"

namespace stkkt {

// Where a block product takes its right-hand sides from: formed already
// (vec, value (col, c) at col vsi + c), or, for one right-hand side, the chunk sums
// of the previous product, base - sum (base == nullptr: the sum), which the
// workgroups of the first row tile then also write to out.
struct ProductInput {
  const double *vec;
  int vsi;
  const double *base, *partial;
  double *out;
  int ld, nch;
};

namespace {

constexpr int kPanel = 64;   // Gauss-Jordan panel width (= GEMM inner dimension)

// ---------------------------------------------------------------------------
// sparse couplings: for every row r = 3 j + a of a level, its 27 spatial
// neighbours i and slots b (81 entries): column index 3 i + b and the value of
// the (dt) block; neighbours outside the mesh have value 0
// ---------------------------------------------------------------------------
__global__ void coupling_rows_kernel(OpDev op, int n, int dt, int32_t *__restrict__ idx, double *__restrict__ val) {
  const int N = op.N;
  for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < 27 * N; q += gridDim.x * blockDim.x) {
    const int j = q / 27, k = q - 27 * j;
    const int jx = j % op.nn[0], jy = (j / op.nn[0]) % op.nn[1], jz = j / (op.nn[0] * op.nn[1]);
    const int dx = k % 3 - 1, dy = (k / 3) % 3 - 1, dz = k / 9 - 1;
    const int ix = jx + dx, iy = jy + dy, iz = jz + dz;
    const bool in = ix >= 0 && ix < op.nn[0] && iy >= 0 && iy < op.nn[1] && iz >= 0 && iz < op.nn[2];
    double blk[9];
    if (in) kkt_block(op, jx, jy, jz, n, dx, dy, dz, dt, blk);
    const int i = in ? ix + op.nn[0] * (iy + op.nn[1] * iz) : 0;
    for (int a = 0; a < 3; ++a)
      for (int b = 0; b < 3; ++b) {
        const long long e = (long long)(3 * j + a) * 81 + 3 * k + b;
        idx[e] = 3 * i + b;
        val[e] = in ? blk[3 * a + b] : 0.0;
      }
  }
}

// the same couplings by column: for every column c = 3 i + b of the block, the
// rows 3 j + a of the 27 neighbours j of i and their values (0 outside the mesh)
__global__ void coupling_cols_kernel(OpDev op, int n, int dt, int32_t *__restrict__ idx, double *__restrict__ val) {
  const int N = op.N;
  for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < 27 * N; q += gridDim.x * blockDim.x) {
    const int i = q / 27, k = q - 27 * i;
    const int ix = i % op.nn[0], iy = (i / op.nn[0]) % op.nn[1], iz = i / (op.nn[0] * op.nn[1]);
    const int dx = k % 3 - 1, dy = (k / 3) % 3 - 1, dz = k / 9 - 1;
    const int jx = ix + dx, jy = iy + dy, jz = iz + dz;
    const bool in = jx >= 0 && jx < op.nn[0] && jy >= 0 && jy < op.nn[1] && jz >= 0 && jz < op.nn[2];
    double blk[9];
    if (in) kkt_block(op, jx, jy, jz, n, -dx, -dy, -dz, dt, blk);
    const int j = in ? jx + op.nn[0] * (jy + op.nn[1] * jz) : 0;
    for (int b = 0; b < 3; ++b)
      for (int a = 0; a < 3; ++a) {
        const long long e = (long long)(3 * i + b) * 81 + 3 * k + a;
        idx[e] = 3 * j + a;
        val[e] = in ? blk[3 * a + b] : 0.0;
      }
  }
}

// S = D_k (column-major, zero before), from the dt = 0 coupling rows: a thread
// per coupling (a row's 81 place their values in 81 different columns, but for
// those outside the mesh, which are 0 and leave no trace).
__global__ void dense_from_rows_kernel(int nb, const int32_t *__restrict__ idx, const double *__restrict__ val,
                                       double *__restrict__ S) {
  for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < 81 * nb; q += gridDim.x * blockDim.x) {
    const double v = val[q];
    if (v != 0.0) S[(long long)idx[q] * nb + q / 81] = v;
  }
}

// the same couplings node by node, for kernels with a thread per node: first
// unknown of neighbour k of node j at node[k N + j] (0 outside the mesh),
// entry (a, b) of its block at val[(9 k + 3 b + a) N + j]
__global__ void coupling_nodes_kernel(OpDev op, int n, int dt, int32_t *__restrict__ node, double *__restrict__ val) {
  const int N = op.N;
  for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < 27 * N; q += gridDim.x * blockDim.x) {
    const int k = q / N, j = q - k * N;
    const int jx = j % op.nn[0], jy = (j / op.nn[0]) % op.nn[1], jz = j / (op.nn[0] * op.nn[1]);
    const int dx = k % 3 - 1, dy = (k / 3) % 3 - 1, dz = k / 9 - 1;
    const int ix = jx + dx, iy = jy + dy, iz = jz + dz;
    const bool in = ix >= 0 && ix < op.nn[0] && iy >= 0 && iy < op.nn[1] && iz >= 0 && iz < op.nn[2];
    double blk[9];
    if (in) kkt_block(op, jx, jy, jz, n, dx, dy, dz, dt, blk);
    node[q] = in ? 3 * (ix + op.nn[0] * (iy + op.nn[1] * iz)) : 0;
    for (int b = 0; b < 3; ++b)
      for (int a = 0; a < 3; ++a) val[(long long)(9 * k + 3 * b + a) * N + j] = in ? blk[3 * a + b] : 0.0;
  }
}

// S(r, c) -= sum_t L(r, idx_t) E(idx_t, c)   (column-major S, E; L rows sparse)
// A thread takes the three rows of a node, which have the same columns idx_t,
// for kSchurCols columns of S at a time: an entry of E serves three products,
// and the tables, laid out for it, are read once per eight columns.  With a
// thread per row, each reading its own 81 table entries one after the other,
// the kernel took 356 us at nb = 2187, now 121.
constexpr int kSchurCols = 8;
__global__ void __launch_bounds__(128) schur_update_kernel(int N, const int32_t *__restrict__ node,
                                                           const double *__restrict__ val,
                                                           const double *__restrict__ E, double *__restrict__ S) {
  const int nb = 3 * N, c0 = blockIdx.y * kSchurCols, nc = min(kSchurCols, nb - c0);
  const double *Ec = E + (long long)c0 * nb;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= N) return;
  double acc[3][kSchurCols];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int q = 0; q < kSchurCols; ++q) acc[a][q] = 0.0;
  for (int k = 0; k < 27; ++k) {
    const int i = node[k * N + j];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const double *v = val + (long long)(9 * k + 3 * b) * N + j;
      const double v0 = v[0], v1 = v[N], v2 = v[2 * N];
#pragma unroll
      for (int q = 0; q < kSchurCols; ++q) {
        const double x = Ec[(long long)(q < nc ? q : 0) * nb + i + b];
        acc[0][q] += v0 * x;
        acc[1][q] += v1 * x;
        acc[2][q] += v2 * x;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < kSchurCols; ++q)
    if (q < nc)
#pragma unroll
      for (int a = 0; a < 3; ++a) S[(long long)(c0 + q) * nb + 3 * j + a] -= acc[a][q];
}

// E(:, c) = sum_t Sinv(:, row_t) U(row_t, c), the rows of column c of U given
// as (row index, value) pairs; the three columns of a node have the same rows,
// so a thread forms the three entries of its row from one read of Sinv (a
// thread per entry took 121 us at nb = 2187, this 72).
__global__ void __launch_bounds__(256) e_from_cols_kernel(int nb, const int32_t *__restrict__ cidx,
                                                          const double *__restrict__ cval,
                                                          const double *__restrict__ Sinv, double *__restrict__ E) {
  const int i = blockIdx.y;
  const cptr<int32_t> idx = as_const(cidx) + 243LL * i;
  const cptr<double> val = as_const(cval) + 243LL * i;
  for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < nb; r += gridDim.x * blockDim.x) {
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;
#pragma unroll 9
    for (int t = 0; t < 81; ++t) {
      const double x = Sinv[(long long)idx[t] * nb + r];
      a0 += val[t] * x;
      a1 += val[81 + t] * x;
      a2 += val[162 + t] * x;
    }
    double *e = E + 3LL * i * nb + r;
    e[0] = a0;
    e[nb] = a1;
    e[2LL * nb] = a2;
  }
}

// ---------------------------------------------------------------------------
// blocked Gauss-Jordan inverse of the n x n row-major buffer A (in place)
// ---------------------------------------------------------------------------
__device__ inline void block_argmax(double v, int i, double *sv, int *si) {
  // largest |v|, smallest index on ties, over the workgroup
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int off = 32; off > 0; off >>= 1) {
    const double ov = __shfl_down(v, off, 64);
    const int oi = __shfl_down(i, off, 64);
    if (ov > v || (ov == v && oi < i)) {
      v = ov;
      i = oi;
    }
  }
  if (lane == 0) {
    sv[w] = v;
    si[w] = i;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < (int)(blockDim.x >> 6); ++k)
      if (sv[k] > sv[0] || (sv[k] == sv[0] && si[k] < si[0])) {
        sv[0] = sv[k];
        si[0] = si[k];
      }
  }
  __syncthreads();
}

// The panel columns [k, k + w) of all rows are eliminated in a column-major
// copy P (P[q * n + i] = A[i][k + q]), so that the pivot search reads a
// column contiguously and the elimination is coalesced across rows.
// Both copies go through a 64 x 64 LDS tile.
__global__ void gje_panel_gather_kernel(int n, int k, int w, const double *__restrict__ A, double *__restrict__ P) {
  __shared__ double tile[64][65];
  const int i0 = blockIdx.x * 64;
  for (int q = threadIdx.x; q < 64 * 64; q += blockDim.x) {
    const int r = q / 64, t = q % 64;
    tile[r][t] = (i0 + r < n && t < w) ? A[(long long)(i0 + r) * n + k + t] : 0.0;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < 64 * 64; q += blockDim.x) {
    const int t = q / 64, r = q % 64;
    if (i0 + r < n && t < w) P[(long long)t * n + i0 + r] = tile[r][t];
  }
}

__global__ void gje_panel_scatter_kernel(int n, int k, int w, const double *__restrict__ P, double *__restrict__ A) {
  __shared__ double tile[64][65];
  const int i0 = blockIdx.x * 64;
  for (int q = threadIdx.x; q < 64 * 64; q += blockDim.x) {
    const int t = q / 64, r = q % 64;
    tile[r][t] = (i0 + r < n && t < w) ? P[(long long)t * n + i0 + r] : 0.0;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < 64 * 64; q += blockDim.x) {
    const int r = q / 64, t = q % 64;
    if (i0 + r < n && t < w) A[(long long)(i0 + r) * n + k + t] = tile[r][t];
  }
}

// Gauss-Jordan step for column c of the panel [k, e), part 1 (one
// workgroup): pivot search over rows >= c, swap of the two rows' panel
// segments (the rest of the rows is swapped once per panel, gje_laswp_kernel;
// swp[c - k] records the pivot row), and the pivot row's panel segment divided
// by the pivot (its column-c entry replaced by 1 first); the segment goes to prow.
__global__ void __launch_bounds__(1024) gje_pivot_kernel(int n, int k, int e, int c, double *__restrict__ P,
                                                         int32_t *__restrict__ piv, int32_t *__restrict__ swp,
                                                         double *__restrict__ prow, double *__restrict__ fcol,
                                                         int *__restrict__ status) {
  __shared__ double sv[16];
  __shared__ int si[16];
  if (*status) return;
  const int j = c - k, w = e - k;
  const double *Pc = P + (long long)j * n;
  double best = -1.0;
  int bi = n;
  for (int i = c + threadIdx.x; i < n; i += blockDim.x) {
    const double v = fabs(Pc[i]);
    if (v > best || (v == best && i < bi)) {
      best = v;
      bi = i;
    }
  }
  block_argmax(best, bi, sv, si);
  const int p = si[0];
  const double pv = sv[0];
  if (!(pv > 0.0) || !std::isfinite(pv)) {
    if (threadIdx.x == 0) *status = 1;
    return;
  }
  if (threadIdx.x == 0) swp[j] = p;
  if (p != c) {
    if ((int)threadIdx.x < w) {
      double *Pq = P + (long long)threadIdx.x * n;
      const double t = Pq[c];
      Pq[c] = Pq[p];
      Pq[p] = t;
    }
    if (threadIdx.x == 0) {
      const int32_t t = piv[c];
      piv[c] = piv[p];
      piv[p] = t;
    }
  }
  __syncthreads();
  // the multipliers of the elimination: column j after the swap
  for (int i = threadIdx.x; i < n; i += blockDim.x) fcol[i] = Pc[i];
  const double a = Pc[c];
  __syncthreads();
  if ((int)threadIdx.x < w) {
    double *Pq = P + (long long)threadIdx.x * n;
    const double v = ((int)threadIdx.x == j ? 1.0 : Pq[c]) / a;
    prow[threadIdx.x] = v;
    Pq[c] = v;
  }
}

// Part 2 (one thread per entry, grid rows x panel columns): eliminate column
// c from every other row of the panel, P[q][i] -= fcol[i] prow[q] (entry
// j = c - k becoming -fcol[i] prow[j]); the multipliers come from the copy
// fcol, so no entry is read after another thread has written it.
__global__ void __launch_bounds__(256) gje_elim_kernel(int n, int k, int c, double *__restrict__ P,
                                                       const double *__restrict__ prow,
                                                       const double *__restrict__ fcol,
                                                       const int *__restrict__ status) {
  if (*status) return;
  const int j = c - k, q = blockIdx.y;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n || i == c) return;
  const double f = fcol[i], pq = prow[q];
  double *x = P + (long long)q * n + i;
  *x = (q == j) ? -f * pq : *x - f * pq;
}

// ---------------------------------------------------------------------------
// The same Gauss-Jordan steps for all columns of a panel in one cooperative
// launch.  Workgroup g keeps the panel segments of rows [g R, g R + R) in LDS
// (column-major, padded: L[t (R + 1) + r]) for the whole panel; step c:
//  1. every workgroup finds its largest |entry| in column c over its rows
//     >= c (smallest row on ties) and publishes it, with that row's segment,
//     in slot (c & 1) of the candidate tables; the owner of row c publishes
//     row c's segment;
//  2. grid barrier;
//  3. every workgroup picks the same pivot row p from the candidates (largest
//     value, smallest row on ties: the choice of gje_pivot_kernel), forms the
//     scaled pivot row and eliminates column c from its own rows; the owner
//     of row p puts row c's old segment in its place (the swap), the owner of
//     row c the scaled pivot row.
// The two candidate slots alternate, so a slot is rewritten only after every
// workgroup has passed the barrier that follows its reads.  The barrier
// counter grows by the number of workgroups per step and is zeroed once per
// inversion; bar0 is the number of steps taken by earlier launches.  A
// barrier that has not completed after `spin_limit` polls (the default is
// about a second) sets the abort flag and status 2, and every workgroup
// leaves at its next barrier, so the launch always ends.
// ---------------------------------------------------------------------------
constexpr int kGjThreads = 1024;
constexpr unsigned kGjSpinLimit = 1u << 20;   // default bound on the polls of one barrier

struct GjSync {
  double *candv;     // [2][nwg] largest |entry|
  int32_t *candi;    // [2][nwg] its row
  double *candrow;   // [2][nwg][kPanel] that row's panel segment
  double *crow;      // [2][kPanel] row c's panel segment
  unsigned *count;   // barrier arrivals
  int *abort;        // set by a barrier that timed out
  unsigned spin_limit;
};

// All threads of the workgroup; false if the barrier was abandoned.  Every
// global write a step makes before its barrier (candidate tables, row c,
// pivot records) comes from wavefront 0, so thread 0's release ordering of its
// arrival covers them; the wait polls with relaxed loads and ends with one
// acquire fence, whose cache invalidation the other wavefronts of the
// compute unit see after the workgroup barrier.
__device__ inline bool gj_grid_barrier(const GjSync &gs, unsigned target) {
  __shared__ int ok;
  __syncthreads();
  if (threadIdx.x == 0) {
    __hip_atomic_fetch_add(gs.count, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    int good = 1;
    unsigned spins = 0;
    while (__hip_atomic_load(gs.count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
      if (__hip_atomic_load(gs.abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 || ++spins > gs.spin_limit) {
        __hip_atomic_store(gs.abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        good = 0;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    ok = good;
  }
  __syncthreads();
  return ok != 0;
}

// loads of values other workgroups wrote during the launch
template <typename T> __device__ inline T ld_agent(const T *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ void gj_reset_kernel(GjSync gs) {
  if (threadIdx.x == 0) {
    *gs.count = 0u;
    *gs.abort = 0;
  }
}

__global__ void __launch_bounds__(kGjThreads) gje_panel_kernel(int n, int k, int e, int R, double *__restrict__ A,
                                                              int32_t *__restrict__ piv, int32_t *__restrict__ swp,
                                                              GjSync gs, unsigned bar0, int *__restrict__ status) {
  extern __shared__ double gj_lds[];
  __shared__ double wv[kGjThreads / 64], prow_s[kPanel], crow_s[kPanel];
  __shared__ int wi[kGjThreads / 64];
  if (*status) return;
  const int tid = threadIdx.x, g = blockIdx.x, nwg = gridDim.x;
  const int w = e - k, LD = R + 1;
  const int r0 = g * R, rows = min(R, n - r0);
  double *L = gj_lds;
  for (int q = tid; q < R * w; q += kGjThreads) {
    const int r = q / w, t = q % w;
    L[t * LD + r] = r < rows ? A[(long long)(r0 + r) * n + k + t] : 0.0;
  }
  __syncthreads();
  // this thread's row and first column in the elimination
  const int rr = tid % R, t0 = tid / R, tstep = kGjThreads / R;
  for (int j = 0; j < w; ++j) {
    const int c = k + j, par = j & 1;
    // 1. local candidate
    double best = -1.0;
    int bi = n;
    for (int r = tid; r < rows; r += kGjThreads) {
      const int i = r0 + r;
      if (i < c) continue;
      const double v = fabs(L[j * LD + r]);
      if (v > best || (v == best && i < bi)) {
        best = v;
        bi = i;
      }
    }
    block_argmax(best, bi, wv, wi);
    {
      const double lv = wv[0];
      const int li = wi[0];
      if (tid == 0) {
        gs.candv[par * nwg + g] = lv;
        gs.candi[par * nwg + g] = li;
      }
      if (tid < w) {
        gs.candrow[((long long)par * nwg + g) * kPanel + tid] = li < n ? L[tid * LD + (li - r0)] : 0.0;
        if (c >= r0 && c < r0 + rows) gs.crow[par * kPanel + tid] = L[tid * LD + (c - r0)];
      }
    }
    // 2. all candidates published
    if (!gj_grid_barrier(gs, (unsigned)nwg * (bar0 + (unsigned)j + 1u))) {
      if (tid == 0) __hip_atomic_store(status, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    // 3. the pivot
    {
      double v = -1.0;
      int i = n;
      for (int q = tid; q < nwg; q += kGjThreads) {
        const double cv = ld_agent(gs.candv + par * nwg + q);
        const int ci = ld_agent(gs.candi + par * nwg + q);
        if (cv > v || (cv == v && ci < i)) {
          v = cv;
          i = ci;
        }
      }
      block_argmax(v, i, wv, wi);
    }
    const double pv = wv[0];
    const int p = wi[0];
    if (!(pv > 0.0) || !std::isfinite(pv)) {
      if (tid == 0) *status = 1;
      return;
    }
    const int gp = p / R;
    if (tid < w) {
      const double a = ld_agent(gs.candrow + ((long long)par * nwg + gp) * kPanel + j);
      const double x = ld_agent(gs.candrow + ((long long)par * nwg + gp) * kPanel + tid);
      prow_s[tid] = (tid == j ? 1.0 : x) / a;
      crow_s[tid] = ld_agent(gs.crow + par * kPanel + tid);
    }
    if (g == 0 && tid == 0) {
      swp[j] = p;
      if (p != c) {
        const int32_t t = piv[c];
        piv[c] = piv[p];
        piv[p] = t;
      }
    }
    __syncthreads();
    const int i = r0 + rr;
    const bool valid = rr < rows, isc = i == c, isp = i == p && p != c;
    const double f = valid ? (isp ? crow_s[j] : L[j * LD + rr]) : 0.0;
    __syncthreads();
    if (valid) {
      for (int t = t0; t < w; t += tstep) {
        double nv;
        if (isc) {
          nv = prow_s[t];
        } else {
          const double cur = isp ? crow_s[t] : L[t * LD + rr];
          nv = (t == j) ? -f * prow_s[j] : cur - f * prow_s[t];
        }
        L[t * LD + rr] = nv;
      }
    }
    __syncthreads();
  }
  for (int q = tid; q < R * w; q += kGjThreads) {
    const int r = q / w, t = q % w;
    if (r < rows) A[(long long)(r0 + r) * n + k + t] = L[t * LD + r];
  }
}

// The panel's row swaps, in order, on the columns outside the panel (one
// thread per column).  Skipped after a failed pivot (swp is then incomplete).
__global__ void gje_laswp_kernel(int n, int k, int e, double *__restrict__ A, const int32_t *__restrict__ swp,
                                 const int *__restrict__ status) {
  if (*status) return;
  for (int col = blockIdx.x * blockDim.x + threadIdx.x; col < n; col += gridDim.x * blockDim.x) {
    if (col >= k && col < e) continue;
    for (int c = k; c < e; ++c) {
      const int p = swp[c - k];
      if (p == c) continue;
      const double t = A[(long long)c * n + col];
      A[(long long)c * n + col] = A[(long long)p * n + col];
      A[(long long)p * n + col] = t;
    }
  }
}

// Copy the panel rows [k, e) outside the panel columns: R[t][col] = A[k+t][col]
__global__ void gje_copy_rows_kernel(int n, int k, int e, const double *__restrict__ A, double *__restrict__ R) {
  const int t = blockIdx.y;
  for (int col = blockIdx.x * blockDim.x + threadIdx.x; col < n; col += gridDim.x * blockDim.x)
    R[(long long)t * n + col] = (col >= k && col < e) ? 0.0 : A[(long long)(k + t) * n + col];
}

// Trailing update outside the panel columns, a rank-(e - k) product:
//   rows outside the panel:  A[i][col] += sum_t A[i][k+t] R[t][col]
//   panel rows:              A[i][col]  = sum_t A[i][k+t] R[t][col]
// on the FP64 matrix cores (v_mfma_f64_16x16x4: lane l supplies a = A[l%16][l/16]
// and b = B[l/16][l%16] and holds D[l/16 + 4r][l%16], r = 0..3).  A workgroup
// of 8 wavefronts owns a 64 x 128 output tile; wavefront (wr, wc) a 32 x 32
// part of it, as 2 x 2 blocks of 16 x 16.  The accumulators start from the
// tile's current values (0 for panel rows); the panel is taken in two passes of
// 32 columns, each staging the A panel slice (64 rows x 32) and the R slice
// (32 x 128) in LDS, padded so that a wavefront's operand read meets every bank
// twice.  All of the tile's loads but the second pass's are requested together
// and those before the first pass's products.  About 54 KB of LDS and at most
// 128 registers let two workgroups share a compute unit.  A 128 x 128 tile
// leaves 324 tiles on 256 compute units at n = 2187, so that some take two: 38
// us for the whole update against 29.
constexpr int kUpdRows = 64;
constexpr int kUpdTile = 128;
constexpr int kUpdThreads = 512;
constexpr int kUpdK = 32;
constexpr int kUpdLdA = kUpdK + 2, kUpdLdR = kUpdTile + 16;
constexpr size_t kUpdLds = sizeof(double) * ((size_t)kUpdRows * kUpdLdA + (size_t)kUpdK * kUpdLdR);
typedef double f64x4 __attribute__((ext_vector_type(4)));

// The tile at (row0, col0): out = A outside the panel rows, 0 inside them, plus
// A[:][k + t] rrow(t)[:] over the panel, for the columns `mine` accepts; the
// columns `copied` accepts go from A to out unchanged.  A may be out: a tile
// then reads its own entries before it writes them, and no tile writes the
// panel columns.
template <typename Mine, typename Copied, typename Row>
__device__ inline void update_tile(int n, int k, int e, int row0, int col0, const double *A, double *out, Mine mine,
                                   Copied copied, Row rrow) {
  extern __shared__ double upd_lds[];
  double(*As)[kUpdLdA] = reinterpret_cast<double(*)[kUpdLdA]>(upd_lds);                        // [row][t]
  double(*Rs)[kUpdLdR] = reinterpret_cast<double(*)[kUpdLdR]>(upd_lds + kUpdRows * kUpdLdA);   // [t][col]
  const int w = e - k;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave >> 2, wc = wave & 3;
  const int li = lane & 15, lk = lane >> 4;
  constexpr int kA = kUpdRows * kUpdK / kUpdThreads, kR = kUpdK * kUpdTile / kUpdThreads;
  constexpr int kRowsA = kUpdThreads / kUpdK, kRowsR = kUpdThreads / kUpdTile;   // rows of one round of loads
  double ra[kA], rr[kR];
  const int at = tid % kUpdK, ar = tid / kUpdK, rc = tid % kUpdTile;
  const int rt = __builtin_amdgcn_readfirstlane(tid / kUpdTile);   // a wavefront stays in one row
  auto request = [&](int kb) {
#pragma unroll
    for (int u = 0; u < kA; ++u) {
      const int i = row0 + ar + u * kRowsA;
      ra[u] = (i < n && kb + at < w) ? A[(long long)i * n + k + kb + at] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < kR; ++u) {
      const int t = kb + rt + u * kRowsR, col = col0 + rc;
      rr[u] = (t < w && col < n && !copied(col)) ? rrow(t)[col] : 0.0;
    }
  };
  auto stage = [&]() {
#pragma unroll
    for (int u = 0; u < kA; ++u) As[ar + u * kRowsA][at] = ra[u];
#pragma unroll
    for (int u = 0; u < kR; ++u) Rs[rt + u * kRowsR][rc] = rr[u];
  };
  if (w > 0) request(0);
  f64x4 acc[2][2];
#pragma unroll
  for (int bi = 0; bi < 2; ++bi)
#pragma unroll
    for (int bj = 0; bj < 2; ++bj) {
      const int col = col0 + wc * 32 + bj * 16 + li;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = row0 + wr * 32 + bi * 16 + lk + 4 * r;
        const bool acc_row = i < n && mine(col) && (!(i >= k && i < e) || copied(col));
        acc[bi][bj][r] = acc_row ? A[(long long)i * n + col] : 0.0;
      }
    }
  for (int kb = 0; kb < w; kb += kUpdK) {
    if (kb > 0) __syncthreads();
    stage();
    __syncthreads();
    if (kb + kUpdK < w) request(kb + kUpdK);
#pragma unroll
    for (int t0 = 0; t0 < kUpdK; t0 += 4) {
      double a[2], b[2];
#pragma unroll
      for (int bi = 0; bi < 2; ++bi) a[bi] = As[wr * 32 + bi * 16 + li][t0 + lk];
#pragma unroll
      for (int bj = 0; bj < 2; ++bj) b[bj] = Rs[t0 + lk][wc * 32 + bj * 16 + li];
#pragma unroll
      for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
          acc[bi][bj] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[bi], b[bj], acc[bi][bj], 0, 0, 0);
    }
  }
#pragma unroll
  for (int bi = 0; bi < 2; ++bi)
#pragma unroll
    for (int bj = 0; bj < 2; ++bj) {
      const int col = col0 + wc * 32 + bj * 16 + li;
      if (!mine(col)) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = row0 + wr * 32 + bi * 16 + lk + 4 * r;
        if (i >= n) continue;
        out[(long long)i * n + col] = acc[bi][bj][r];
      }
    }
}

__global__ void __launch_bounds__(kUpdThreads, 4) gje_update_kernel(int n, int k, int e, int cb, int ce, int xb,
                                                                    int xe, int ct0, double *A,
                                                                    const double *__restrict__ R) {
  // columns this launch updates
  auto mine = [&](int col) {
    return col >= cb && col < ce && col < n && !(col >= k && col < e) && !(col >= xb && col < xe);
  };
  update_tile(n, k, e, (int)blockIdx.y * kUpdRows, (ct0 + (int)blockIdx.x) * kUpdTile, A, A, mine,
              [](int) { return false; }, [&](int t) { return R + (long long)t * n; });
}

// Elimination with the pivots searched among each panel's own rows (block
// pivoting).  The Schur blocks of the coarse solve need no row exchanges
// across panels: with the pivots restricted to each 64-row diagonal block the
// inverse agrees with partial pivoting over all rows to about 1e-14 (and with
// LAPACK's inverse), so a panel needs no device-wide exchange per column, and
// one launch takes the matrix from panel to panel.  It reads `O` and writes
// `N` (the two exchange their places for the next launch, so that nothing it
// reads is overwritten and the panel's rows need no copy of their own):
//
// The first npan workgroups take the panel K = [k, e), w = e - k <= 64, to its
// multipliers.  Workgroup g (eight wavefronts) owns the rows [64 g, 64 g + 64):
//  1. brings the diagonal block D = O[K][K] (each workgroup for itself) and its
//     own rows' panel columns up to date with the previous panel [kp, ep) (none
//     when kp == ep): two 64 x 64 x 64 products on the matrix cores, with all
//     their loads requested up front;
//  2. inverts D in LDS, sixteen columns at a time: the first wavefront holds
//     them in registers (lane r: row r).  Step j takes the pivot row p of column
//     j among the rows not yet used (the largest |entry|, the smallest row on
//     ties: a lane reduction over the high words, and one over the low words
//     where several rows have the same) and eliminates column j from its
//     sixteen columns.  All wavefronts then bring the other 48 columns up to
//     date with a rank-16 product.  Rows are not exchanged: row p_j of the
//     result is row j of (P D)^{-1}, P the order of the pivots;
//  3. writes -(its panel segment) (P D)^{-1} into N (one more product), the
//     workgroup that owns K (P D)^{-1} itself, and perm and the panel's
//     entries of piv.
// Every workgroup inverts the same block to the same bits.  A zero or
// non-finite pivot sets *failed, and later launches do nothing: the word that a
// launch tests is the one its predecessor wrote and nobody writes meanwhile, so
// that all wavefronts of all its workgroups decide alike (they share barriers
// and the order of the pivots in LDS).
//
// The other workgroups update the tiles of all columns outside K by the
// previous panel, whose rows are read in the order of its pivots (permp); its
// own columns are copied.
//
// The inversion is a serial chain and bounds the launch: 25 of the panel's 37
// us at n = 2187, 64 pivot steps of about 0.3 us with four rank-16 products
// between them (8 us for the loads and products before); the launch takes 43
// us, the update's tiles beside the panel.  Held in
// one wavefront's registers a step needs no barrier and no LDS.  Spread over
// the eight wavefronts, with launches of their own for the update (on a second
// stream) and for the panel's rows, a panel took 81 us; with the own rows'
// operands staged in LDS after the diagonal block's, the loads took 16 us.
constexpr int kBpThreads = 512;
constexpr int kBpCols = 16;   // columns eliminated in one wavefront's registers
constexpr int kBpLd = kPanel + 1;
constexpr size_t kBpLds = sizeof(double) * 2 * (size_t)kPanel * kBpLd;
// LDS of a launch.  While the update is hidden beside the panel, the panel's
// workgroups get compute units of their own (more than half of the LDS each):
// n = 2187 (630 tiles) 52.0 us a panel against 53.1 with two workgroups per
// compute unit, which wait for each other's matrix instructions.  Where the
// update takes longer than the panel two are better: n = 3993 (2016 tiles) 93
// against 111 us.
constexpr size_t kStepLdsTwo = kBpLds > kUpdLds ? kBpLds : kUpdLds, kStepLdsOne = 84 * 1024;
constexpr int kStepOneTiles = 3 * 256;
static_assert(kBpThreads == kUpdThreads, "one launch holds both kinds of workgroup");

// largest value over the wavefront's lanes
__device__ inline unsigned wave_max_u32(unsigned v) {
  auto step = [&v](unsigned o) { v = o > v ? o : v; };
  step((unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));   // row_shr:1
  step((unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));   // row_shr:2
  step((unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));   // row_shr:4
  step((unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));   // row_shr:8
  step((unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));   // row_bcast:15
  step((unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));   // row_bcast:31
  return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}

__device__ inline double lane_value(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// 64 x 64 product on the eight wavefronts of the workgroup: wavefront v
// forms the 16 x 16 blocks (v / 2, 2 (v % 2)) and the one right of it.
__device__ inline void bp_product(const double *X, const double *Y, f64x4 (&acc)[2]) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4, bi = wv >> 1, bj = 2 * (wv & 1);
#pragma unroll 4
  for (int t0 = 0; t0 < kPanel; t0 += 4) {
    const double a = X[(16 * bi + li) * kBpLd + t0 + lk];
#pragma unroll
    for (int u = 0; u < 2; ++u)
      acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, Y[(t0 + lk) * kBpLd + 16 * (bj + u) + li], acc[u], 0, 0, 0);
  }
}

__device__ inline void panel_rows_step(int n, int kp, int ep, int k, int e, const double *__restrict__ O,
                                       double *__restrict__ N, const int32_t *__restrict__ permp,
                                       int32_t *__restrict__ perm, int32_t *__restrict__ piv,
                                       int *__restrict__ failed) {
  extern __shared__ double upd_lds[];
  __shared__ int step_of[kPanel], row_of[kPanel];   // the step that took a row as its pivot row, and the reverse
  double *Sa = upd_lds, *Sb = Sa + kPanel * kBpLd;
  const int w = e - k, wp = ep - kp;
  const int tid = (int)threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4, bi = wv >> 1, bj = 2 * (wv & 1);
  const int i0 = (int)blockIdx.x * kPanel;
  __builtin_amdgcn_s_setprio(3);   // ahead of the tiles that share the compute unit
  // 1. An entry (row, col) of a 16 x 16 block (br, bc) sits in register r of
  // lane (li, lk): row 16 br + lk + 4 r, column 16 bc + li.
  constexpr int kPer = kPanel * kPanel / kBpThreads, kBpWaves = kBpThreads / 64;
  // (a panel with a successor has 64 columns: wp is 0 or 64)
  // loads by 32-bit byte offsets from a row's start, clamped into the matrix
  auto at = [n](const double *base, int row, int col) {
    return *reinterpret_cast<const double *>(reinterpret_cast<const char *>(base) +
                                             (unsigned)sizeof(double) * (unsigned)(row * n + col));
  };
  if (wp > 0) {
    const cptr<int32_t> pp = as_const(permp);
    double d[kPer], x[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {   // a wavefront takes whole rows
      const int a = wv + u * kBpWaves;
      d[u] = at(O + (long long)k * n + kp, min(a, w - 1), lane);
      x[u] = at(O + (long long)kp * n + k, pp[a], min(lane, w - 1));
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int a = wv + u * kBpWaves;
      Sb[a * kBpLd + lane] = a < w ? d[u] : 0.0;
      Sa[a * kBpLd + lane] = lane < w ? x[u] : 0.0;
    }
  }
  f64x4 dia[2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int q = 16 * bi + lk + 4 * r, c = 16 * (bj + u) + li;
      const double v = at(O + (long long)k * n + k, min(q, w - 1), min(c, w - 1));
      dia[u][r] = q < w && c < w ? v : q == c ? 1.0 : 0.0;
    }
  // own rows: the panel's columns, and the previous panel's as operands
  const int rlast = n - 1 - i0;
  double oa[kPanel / 4];
  f64x4 own[2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int c = 16 * (bj + u) + li;
      const double v = at(O + (long long)i0 * n + k, min(16 * bi + lk + 4 * r, rlast), min(c, w - 1));
      own[u][r] = c < w && !(wp > 0 && i0 == kp) ? v : 0.0;   // the previous panel's rows start from 0
    }
  if (wp > 0) {
#pragma unroll
    for (int t = 0; t < kPanel / 4; ++t)
      oa[t] = at(O + (long long)i0 * n + kp, min(16 * bi + li, rlast), 4 * t + lk);
    __syncthreads();
    bp_product(Sb, Sa, dia);
#pragma unroll
    for (int t = 0; t < kPanel / 4; ++t)
#pragma unroll
      for (int u = 0; u < 2; ++u)
        own[u] =
            __builtin_amdgcn_mfma_f64_16x16x4f64(oa[t], Sa[(4 * t + lk) * kBpLd + 16 * (bj + u) + li], own[u], 0, 0, 0);
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int q = 16 * bi + lk + 4 * r, c = 16 * (bj + u) + li;
      Sa[q * kBpLd + c] = own[u][r];
      Sb[q * kBpLd + c] = dia[u][r];
    }
  __syncthreads();
  // 2. (P D)^{-1}; rows and columns past w are those of the identity
  int myq = -1;   // (first wavefront) the step that took this lane's row as its pivot row
  if (wv == 0) step_of[lane] = -1;
#pragma unroll 1
  for (int b0 = 0; b0 < kPanel; b0 += kBpCols) {
    if (wv == 0) {
      double m[kBpCols];
#pragma unroll
      for (int c = 0; c < kBpCols; ++c) m[c] = Sb[lane * kBpLd + b0 + c];
#pragma unroll
      for (int jj = 0; jj < kBpCols; ++jj) {
        // high word of |entry| above those of the rows used already
        const unsigned key = myq < 0 ? (unsigned)__double2hiint(m[jj]) | 0x80000000u : 0u;
        const unsigned top = wave_max_u32(key);
        unsigned long long cand = __ballot(key == top);
        if (cand & (cand - 1)) {
          const unsigned lo = key == top ? (unsigned)__double2loint(m[jj]) : 0u;
          cand &= __ballot(lo == wave_max_u32(lo));
        }
        const int p = (int)__builtin_ctzll(cand);
        const double a = lane_value(m[jj], p), inv = 1.0 / a;
        if (lane == 0 && (!(fabs(a) > 0.0) || !std::isfinite(a))) *failed = 1;
        const bool isp = lane == p;
        const double g = isp ? inv : -m[jj] * inv;
        if (isp) myq = b0 + jj;
#pragma unroll
        for (int u = 1; u < kBpCols; ++u) {   // column jj + 1 first: the next step waits for it
          const int c = (jj + u) % kBpCols;
          const double x = lane_value(m[c], p);
          m[c] = __builtin_fma(g, x, isp ? 0.0 : m[c]);
        }
        m[jj] = g;
      }
#pragma unroll
      for (int c = 0; c < kBpCols; ++c) Sb[lane * kBpLd + b0 + c] = m[c];
      if (myq >= b0) {
        step_of[lane] = myq;
        row_of[myq] = lane;
      }
    }
    __syncthreads();
    // the other column blocks: 4 x 3 tiles of 16 x 16 on eight wavefronts
    f64x4 t[2];
    auto tile = [&](int u, int &br, int &bc) {
      const int q = wv + 8 * u;
      br = q & 3;
      bc = q >> 2;
      bc += bc >= b0 / kBpCols;
      return q < 12;
    };
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      int br, bc;
      if (!tile(u, br, bc)) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * br + lk + 4 * r;
        t[u][r] = step_of[row] >= b0 ? 0.0 : Sb[row * kBpLd + 16 * bc + li];
      }
#pragma unroll
      for (int s0 = 0; s0 < kBpCols; s0 += 4)
        t[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(Sb[(16 * br + li) * kBpLd + b0 + s0 + lk],
                                                    Sb[row_of[b0 + s0 + lk] * kBpLd + 16 * bc + li], t[u], 0, 0, 0);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      int br, bc;
      if (!tile(u, br, bc)) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) Sb[(16 * br + lk + 4 * r) * kBpLd + 16 * bc + li] = t[u][r];
    }
    __syncthreads();
  }
  {
    // the rows in the order of the pivots
    double v[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) v[u] = Sb[lane * kBpLd + kPer * wv + u];
    const int q = max(step_of[lane], 0);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPer; ++u) Sb[q * kBpLd + kPer * wv + u] = v[u];
  }
  __syncthreads();
  // 3. the multipliers; panels and row groups are both 64 wide, so one
  // workgroup owns exactly the panel's rows
  if (i0 == k) {
    for (int q = tid; q < kPanel * kPanel; q += kBpThreads) {
      const int a = q / kPanel, b = q % kPanel;
      if (a < w && b < w) N[(long long)(k + a) * n + k + b] = Sb[a * kBpLd + b];
    }
    if (wv == 0) {
      const bool real = lane < w && myq >= 0 && myq < w;   // (a row past w is a pivot row of a singular block only)
      const int32_t old = real ? piv[k + lane] : 0;
      if (real) {
        piv[k + myq] = old;
        perm[myq] = lane;
      }
    }
    return;
  }
#pragma unroll
  for (int u = 0; u < 2; ++u) dia[u] = f64x4{0.0, 0.0, 0.0, 0.0};
  bp_product(Sa, Sb, dia);
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = i0 + 16 * bi + lk + 4 * r, c = 16 * (bj + u) + li;
      if (i < n && c < w) N[(long long)i * n + k + c] = -dia[u][r];
    }
}

__global__ void __launch_bounds__(kBpThreads, 4) gje_block_step_kernel(int n, int npan, int kp, int ep, int k, int e,
                                                                       const double *__restrict__ O,
                                                                       double *__restrict__ N,
                                                                       const int32_t *__restrict__ permp,
                                                                       int32_t *__restrict__ perm,
                                                                       int32_t *__restrict__ piv,
                                                                       const int *__restrict__ failed_before,
                                                                       int *__restrict__ failed) {
  if (*failed_before) {   // permp is then incomplete
    if (blockIdx.x == 0 && threadIdx.x == 0) *failed = 1;
    return;
  }
  if ((int)blockIdx.x < npan) {
    panel_rows_step(n, kp, ep, k, e, O, N, permp, perm, piv, failed);
    return;
  }
  const int nt = (n + kUpdTile - 1) / kUpdTile, t = (int)blockIdx.x - npan;
  update_tile(n, kp, ep, (t / nt) * kUpdRows, (t % nt) * kUpdTile, O, N,
              [&](int col) { return col < n && !(col >= k && col < e); },
              [&](int col) { return col >= kp && col < ep; },
              [&](int a) { return O + (long long)(kp + permp[a]) * n; });
}

// out[i][piv[j]] = A[i][j]
__global__ void gje_unpermute_kernel(int n, const double *__restrict__ A, const int32_t *__restrict__ piv,
                                     double *__restrict__ out) {
  const int i = blockIdx.y;
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < n; j += gridDim.x * blockDim.x)
    out[(long long)i * n + piv[j]] = A[(long long)i * n + j];
}

__global__ void iota_kernel(int n, int32_t *p) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = i;
}

// ---------------------------------------------------------------------------
// application
// ---------------------------------------------------------------------------
// A block product leaves its sums over column chunks, partial[(chunk q + c) ld
// + row] for right-hand side c < q.  With one right-hand side and small blocks
// the next launch adds them where it needs them, in chunk order, so no launch of
// its own does only that: a level of the forward sweep is two launches, of the
// backward sweep one.  Every workgroup of a product then adds the sums of its
// columns, rows / 64 times the reads of a separate sum, and a row of couplings
// those of 81: against the block's bytes that grows with nb, and so the added
// form ends at fold_rows().  Both sweeps, separate / added:
//   levels          7           7           9           7           7           5
//   nb           1029        1536        2187        3000        3993        6591
//   GEMV    119 / 108   119 / 102   206 / 190   200 / 202   257 / 285   376 / 490 us
//   MFMA    120 / 120   155 / 159   276 / 296   286 / 329   403 / 506   607 / 656 us
// (GEMV: FP32 blocks, MFMA here: FP64).  Several right-hand sides always keep the
// separate sum (gemm_reduce_kernel): at nb = 2187 and six of them the added form
// took 1300 us a correction against 1045.  The order of the sums is the same.
constexpr int fold_rows(bool gemv) { return gemv ? 2560 : 1280; }

__device__ inline double chunk_sum(const double *__restrict__ partial, int ld, int nch, int row) {
  double s = 0.0;
#pragma unroll 6
  for (int k = 0; k < nch; ++k) s += partial[(long long)k * ld + row];
  return s;
}

// t[i] = r[i] - (L y)[i], y the chunk sums of `partial`, which also go to y;
// with partial == nullptr: t = r.  One wavefront per row: its 81 couplings
// spread over the lanes and summed in a fixed order.
__global__ void __launch_bounds__(256) lower_rhs_kernel(int nb, int ld, int nch, const int32_t *__restrict__ idx,
                                                        const double *__restrict__ val, const double *__restrict__ r,
                                                        const double *__restrict__ partial, double *__restrict__ y,
                                                        double *__restrict__ t, int tsi) {
  const int lane = threadIdx.x & 63;
  for (int i = blockIdx.x * 4 + (threadIdx.x >> 6); i < nb; i += gridDim.x * 4) {
    double s = 0.0;
    if (partial) {
      const long long b = (long long)i * 81;
      // lanes 17..63 of the second round: lane 17 forms the row's own y
      const int j1 = lane < 81 - 64 ? idx[b + 64 + lane] : i;
      const double v0 = val[b + lane], v1 = lane < 81 - 64 ? val[b + 64 + lane] : 0.0;
      const double y0 = chunk_sum(partial, ld, nch, idx[b + lane]);
      const double y1 = lane <= 81 - 64 ? chunk_sum(partial, ld, nch, j1) : 0.0;
      if (lane == 81 - 64) y[i] = y1;
      s = v0 * y0;
      if (lane < 81 - 64) s += v1 * y1;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    }
    if (lane == 0) t[(long long)i * tsi] = r[i] - s;
  }
}

// The same for q right-hand sides with y_c = y + c ldy formed (nullptr: t = r):
// t[i tsi + c] = r_c[i] - (L y_c)[i], the couplings read once for VECS of them
// (blockIdx.y: which), whose values are in flight together.  Bound by the
// latency of the reads: at nb = 1536 sixteen vectors take 7 us, one after the
// other 16, with a wavefront for each 9 (nb = 6591: 18, 23 and 30 us).
template <int VECS>
__global__ void __launch_bounds__(256) lower_rhs_multi_kernel(int nb, int q, const int32_t *__restrict__ idx,
                                                              const double *__restrict__ val,
                                                              const double *__restrict__ r, long long ldr,
                                                              const double *__restrict__ y, long long ldy,
                                                              double *__restrict__ t, int tsi) {
  const int lane = threadIdx.x & 63, c0 = blockIdx.y * VECS, nc = min(VECS, q - c0);
  for (int i = blockIdx.x * 4 + (threadIdx.x >> 6); i < nb; i += gridDim.x * 4) {
    const long long b = (long long)i * 81;
    const bool two = lane < 81 - 64;
    const int i0 = idx[b + lane], i1 = two ? idx[b + 64 + lane] : 0;
    const double v0 = val[b + lane], v1 = two ? val[b + 64 + lane] : 0.0;
    double y0[VECS], y1[VECS], rc[VECS];
#pragma unroll
    for (int c = 0; c < VECS; ++c) {
      const int cc = c0 + min(c, nc - 1);
      y0[c] = y ? y[cc * ldy + i0] : 0.0;
      y1[c] = y && two ? y[cc * ldy + i1] : 0.0;
      rc[c] = r[cc * ldr + i];
    }
#pragma unroll
    for (int c = 0; c < VECS; ++c) {
      double s = 0.0;
      if (y) {
        s = v0 * y0[c];
        if (two) s += v1 * y1[c];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
      }
      if (lane == 0 && c < nc) t[(long long)i * tsi + c0 + c] = rc[c] - s;
    }
  }
}

// entry col of the one right-hand side
__device__ inline double product_input(const ProductInput &in, int col, bool write) {
  if (in.vec) return in.vec[(long long)col * in.vsi];
  const double s = chunk_sum(in.partial, in.ld, in.nch, col);
  const double v = in.base ? in.base[col] - s : s;
  if (write) in.out[col] = v;
  return v;
}

// Y = A X, one vector, FP32 blocks: a wavefront owns 64 rows and a chunk of
// kGvCols columns, one row per lane; partial[chunk][row] = sum over the
// chunk's columns in FP32, ascending.  AHEAD columns are in flight per
// wavefront: 64 (16 KB) up to fold_rows(), where the chip has few wavefronts (nb =
// 2187: 19 MB of a block in 7.4 us, 18 us with 256-row workgroups and the loads
// left to the compiler), 32 above (nb = 6591, both sweeps: 536 to 542 us, 545
// to 547 with 64).
constexpr int kGvRows = 64, kGvCols = 128;

template <int AHEAD>
__global__ void __launch_bounds__(kGvRows) gemv_partial_kernel(int nb, int ld, const float *__restrict__ A,
                                                               ProductInput in, double *__restrict__ partial) {
  static_assert(kGvCols % AHEAD == 0, "whole batches");
  __shared__ float xs[kGvCols];
  const int c0 = blockIdx.y * kGvCols, nc = min(kGvCols, nb - c0);
  const int r = blockIdx.x * kGvRows + (int)threadIdx.x;   // < ld
  const float *a = A + (long long)c0 * ld + r;
  float v[AHEAD];
#pragma unroll
  for (int k = 0; k < AHEAD; ++k) v[k] = a[(long long)min(k, nc - 1) * ld];
  for (int k = threadIdx.x; k < kGvCols; k += kGvRows)
    xs[k] = k < nc ? (float)product_input(in, c0 + k, blockIdx.x == 0) : 0.0f;
  __syncthreads();
  float acc = 0;
#pragma unroll
  for (int b = 0; b < kGvCols; b += AHEAD) {
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) {
      const float u = v[k];
      if (b + AHEAD < kGvCols) v[k] = a[(long long)min(b + AHEAD + k, nc - 1) * ld];
      acc = __builtin_fmaf(u, xs[b + k], acc);   // columns past the chunk count zero times
    }
  }
  if (r < nb) partial[(long long)blockIdx.y * nb + r] = (double)acc;
}

// out = base - chunk sums (base == nullptr: the sums): the end of a sweep.
__global__ void product_finish_kernel(int nb, ProductInput in) {
  for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < nb; r += gridDim.x * blockDim.x)
    product_input(in, r, true);
}

// out_c[r] = base_c[r] - sum_chunks partial[chunk][c][r] (fixed order; base ==
// nullptr: the sum), c = blockIdx.y; the same value also goes to outT[r][c]
__global__ void gemm_reduce_kernel(int nb, int ld, int q, int nchunk, const double *__restrict__ partial,
                                   const double *base, long long ldb, double *out, long long ldo,
                                   double *__restrict__ outT, int tsi) {
  const int c = blockIdx.y;
  for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < nb; r += gridDim.x * blockDim.x) {
    double s = 0.0;
#pragma unroll 8
    for (int k = 0; k < nchunk; ++k) s += partial[((long long)k * q + c) * ld + r];
    const double v = base ? base[c * ldb + r] - s : s;
    out[c * ldo + r] = v;
    outT[(long long)r * tsi + c] = v;
  }
}

// out (leading dimension ld, rows nb..ld-1 zero) = S (nb x nb, leading dimension nb), column c = blockIdx.y
template <typename T>
__global__ void store_padded_kernel(int nb, int ld, const double *__restrict__ S, T *__restrict__ out) {
  const int c = blockIdx.y;
  for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < ld; r += gridDim.x * blockDim.x)
    out[(long long)c * ld + r] = r < nb ? (T)S[(long long)c * nb + r] : (T)0;
}

// ---------------------------------------------------------------------------
// several right-hand sides at once: the product input lies transposed, [column]
// [right-hand side], so that the matrix-core operands of 4 consecutive columns
// are one contiguous read.  Staged in LDS first, as the form with chunk sums
// does, a product of sixteen took 56 us at nb = 6591 in FP32, now 42.
// ---------------------------------------------------------------------------
constexpr int kMrRows = 64, kMrRhs = 16, kMrThreads = 256, kMrAhead = 8;

// Y = A X for up to 16 right-hand sides on the FP64 matrix cores
// (v_mfma_f64_16x16x4: lane l supplies a = A[l%16][l/16], b = B[l/16][l%16]
// and holds D[l/16 + 4j][l%16], j = 0..3).  A workgroup of 4 wavefronts owns
// 64 rows and a chunk of columns (blockIdx.y); step s of wavefront w takes
// columns 16 s + 4 w .. 16 s + 4 w + 3 of the chunk.  Lane (i, kk) =
// (l%16, l/16) reads rows 4i .. 4i + 3 of its column with one 16-byte load
// (float) or two (double) and gives row 4i + m to product m (m = 0..3), so
// product m covers rows m, 4 + m, .., 60 + m of the tile and each column of
// the tile is one contiguous 256- or 512-byte read.  Loads run kMrAhead steps
// ahead of the products, with no branch: a column past the chunk reads the
// chunk's last column and enters as zero.  The four wavefronts' sums
// are added in LDS and written to partial[chunk][c][row] (leading dimension
// ld).  Float blocks are widened to double on load.  Column n of a product
// depends on column n of X only, so a right-hand side's result does not
// depend on the others.
// raw loads of 4 rows, widened and masked only when the products use them
// (a conversion right after the load would make the wavefront wait for it)
struct Rows4f {
  float4 v;
  __device__ void load(const float *p) { v = *reinterpret_cast<const float4 *>(p); }
  __device__ void get(bool ok, double a[4]) const {
    a[0] = ok ? (double)v.x : 0.0;
    a[1] = ok ? (double)v.y : 0.0;
    a[2] = ok ? (double)v.z : 0.0;
    a[3] = ok ? (double)v.w : 0.0;
  }
};
struct Rows4d {
  double2 u, v;
  __device__ void load(const double *p) {
    u = *reinterpret_cast<const double2 *>(p);
    v = *reinterpret_cast<const double2 *>(p + 2);
  }
  __device__ void get(bool ok, double a[4]) const {
    a[0] = ok ? u.x : 0.0;
    a[1] = ok ? u.y : 0.0;
    a[2] = ok ? v.x : 0.0;
    a[3] = ok ? v.y : 0.0;
  }
};
template <typename T> struct Rows4;
template <> struct Rows4<float> { using type = Rows4f; };
template <> struct Rows4<double> { using type = Rows4d; };

constexpr int kMrBatch = 16 * kMrAhead;   // columns of one load batch (128)

// BATCHES x 128 columns per chunk: a batch's loads are all in flight together,
// the next batch's are issued as the current one is multiplied.  SUMS: the one
// right-hand side is formed (from chunk sums, mostly) into LDS first; else the
// formed right-hand sides are read as operands, beside the block's columns.
template <typename T, int BATCHES, bool SUMS>
__global__ void __launch_bounds__(kMrThreads) gemm_partial_kernel(int nb, int ld, const T *__restrict__ A, int q,
                                                                  ProductInput in, double *__restrict__ partial) {
  __shared__ double lds[4 * kMrRhs * kMrRows];   // (the chunk's input), then the wavefronts' sums [wave][rhs][row]
  static_assert(BATCHES * kMrBatch * kMrRhs <= 4 * kMrRhs * kMrRows, "XT fits");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int r0 = blockIdx.x * kMrRows;
  const int cbeg = blockIdx.y * (BATCHES * kMrBatch), ncol = min(nb - cbeg, BATCHES * kMrBatch), last = ncol - 1;
  const int c_lane = 4 * wave + lk;   // column of step 0 in the chunk
  const T *arow = A + (long long)cbeg * ld + r0 + 4 * li;
  const double *brow = in.vec + (long long)cbeg * in.vsi + min(li, q - 1);   // (!SUMS)
  f64x4 acc[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) acc[m] = f64x4{0.0, 0.0, 0.0, 0.0};
  typename Rows4<T>::type raw[kMrAhead];
  double b[kMrAhead];
  auto fetch = [&](int p, int step) {
    const int cc = min(c_lane + 16 * step, last);
    raw[p].load(arow + (long long)cc * ld);
    if (!SUMS) b[p] = brow[cc * in.vsi];
  };
#pragma unroll
  for (int p = 0; p < kMrAhead; ++p) fetch(p, p);
  if (SUMS) {
    // the input, while the first columns are on their way
    for (int k = tid; k < ncol; k += kMrThreads) lds[k * kMrRhs] = product_input(in, cbeg + k, blockIdx.x == 0);
    __syncthreads();
  }
#pragma unroll
  for (int bt = 0; bt < BATCHES; ++bt) {
#pragma unroll
    for (int p = 0; p < kMrAhead; ++p) {
      const int step = bt * kMrAhead + p, cc = c_lane + 16 * step;
      const double bv = SUMS ? lds[min(cc, last) * kMrRhs + li] : b[p];
      double a[4];
      raw[p].get(cc <= last, a);
#pragma unroll
      for (int m = 0; m < 4; ++m) acc[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[m], bv, acc[m], 0, 0, 0);
      if (bt + 1 < BATCHES) fetch(p, step + kMrAhead);
    }
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int j = 0; j < 4; ++j) lds[(wave * kMrRhs + li) * kMrRows + 4 * (lk + 4 * j) + m] = acc[m][j];
  __syncthreads();
  const int rhs = tid >> 4, rl = 4 * (tid & 15);
  if (rhs >= q) return;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int row = r0 + rl + u;
    const double v = lds[(0 * kMrRhs + rhs) * kMrRows + rl + u] + lds[(1 * kMrRhs + rhs) * kMrRows + rl + u] +
                     lds[(2 * kMrRhs + rhs) * kMrRows + rl + u] + lds[(3 * kMrRhs + rhs) * kMrRows + rl + u];
    if (row < nb) partial[((long long)blockIdx.y * q + rhs) * ld + row] = v;
  }
}

}  // namespace

// Pivots among each panel's rows (the default) unless STKKT_COARSE_PIVOT is
// "global" or STKKT_COARSE_PANEL_ROWS selects one of the global-pivoting
// elimination paths below.
static bool block_pivoting() {
  if (std::getenv("STKKT_COARSE_PANEL_ROWS")) return false;
  const char *e = std::getenv("STKKT_COARSE_PIVOT");
  return !(e && e[0] == 'g');
}

// Rows per workgroup of the cooperative panel elimination (64, 128 or 256;
// STKKT_COARSE_PANEL_ROWS overrides, 0 selects the launch-per-column path),
// or 0 if its workgroups cannot all be resident at once.
static int panel_rows(int n) {
  const char *env = std::getenv("STKKT_COARSE_PANEL_ROWS");
  const int forced = env ? std::atoi(env) : -1;
  int dev = 0, cus = 0, coop = 0;
  STKKT_HIP(hipGetDevice(&dev));
  STKKT_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  STKKT_HIP(hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev));
  if (!coop || forced == 0) return 0;
  for (int R : {128, 256, 64}) {
    if (forced > 0 && R != forced) continue;
    const size_t lds = sizeof(double) * (size_t)kPanel * (R + 1);
    STKKT_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&gje_panel_kernel),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    int per_cu = 0;
    STKKT_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, gje_panel_kernel, kGjThreads, lds));
    if ((n + R - 1) / R <= per_cu * cus) return R;
  }
  return 0;
}

// Second stream and events of the panel look-ahead (default priority).
struct LookAhead {
  hipStream_t side = nullptr;
  hipEvent_t rows_ready = nullptr, rest_done = nullptr;
  LookAhead() {
    try {
      STKKT_HIP(hipStreamCreateWithFlags(&side, hipStreamNonBlocking));
      STKKT_HIP(hipEventCreateWithFlags(&rows_ready, hipEventDisableTiming));
      STKKT_HIP(hipEventCreateWithFlags(&rest_done, hipEventDisableTiming));
    } catch (...) {
      release();
      throw;
    }
  }
  ~LookAhead() { release(); }
  void release() {
    if (side) (void)hipStreamSynchronize(side);
    if (rest_done) (void)hipEventDestroy(rest_done);
    if (rows_ready) (void)hipEventDestroy(rows_ready);
    if (side) (void)hipStreamDestroy(side);
    side = nullptr;
    rows_ready = rest_done = nullptr;
  }
  LookAhead(const LookAhead &) = delete;
  LookAhead &operator=(const LookAhead &) = delete;
};

// Explicit inverse of the n x n row-major matrix in A; the inverse ends in A or
// in tmp, n x n scratch (the pointer returned), the other is overwritten.
// rows: 2 x kPanel x n scratch (the rows of two consecutive panels); pan:
// kPanel x n scratch (the launch-per-column path's panel); swp: 2 kPanel int32
// (with block pivoting the pivot orders of two consecutive panels); piv: n
// int32; gs: candidate tables for ceil(n / 64) workgroups; status: two words,
// zero before the first of all calls, one of them not zero after a failure
// (block pivoting alternates them); la: the look-ahead's side stream and events.
static double *gje_invert(int n, double *A, double *tmp, double *rows, double *pan, double *fcol, int32_t *piv,
                       int32_t *swp, double *prow, const GjSync &gs, int *status, const LookAhead &la,
                       hipStream_t s) {
  static bool attr_set = false;
  if (!attr_set) {
    STKKT_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&gje_update_kernel),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)kUpdLds));
    STKKT_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&gje_block_step_kernel),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)kStepLdsOne));
    attr_set = true;
  }
  const bool block = block_pivoting();
  const int R = block ? 0 : panel_rows(n);
  hipLaunchKernelGGL(iota_kernel, dim3(blocks_for(n, 256, 64)), dim3(256), 0, s, n, piv);
  if (R > 0) hipLaunchKernelGGL(gj_reset_kernel, dim3(1), dim3(64), 0, s, gs);
  const int nt = (n + kUpdTile - 1) / kUpdTile, mt = (n + kUpdRows - 1) / kUpdRows;   // tiles
  // rank-(e - k) update of the columns [cb, ce) outside [xb, xe) on stream st
  auto update = [&](int k, int e, int cb, int ce, int xb, int xe, const double *Rk, hipStream_t st) {
    const int t0 = cb / kUpdTile, t1 = (ce + kUpdTile - 1) / kUpdTile;
    hipLaunchKernelGGL(gje_update_kernel, dim3(t1 - t0, mt), dim3(kUpdThreads), kUpdLds, st, n, k, e, cb, ce, xb, xe,
                       t0, A, Rk);
  };
  // the panel's swaps on the other columns, then its rows into Rk
  auto close_panel = [&](int k, int e, double *Rk) {
    hipLaunchKernelGGL(gje_laswp_kernel, dim3(blocks_for(n, 256, 64)), dim3(256), 0, s, n, k, e, A, swp, status);
    hipLaunchKernelGGL(gje_copy_rows_kernel, dim3(blocks_for(n, 256, 64), e - k), dim3(256), 0, s, n, k, e, A, Rk);
  };
  if (block) {
    // One launch per panel: the previous panel's update beside the panel.  The
    // first only copies beside panel 0, the last only updates (and hands on a
    // failure, so that the next call finds it in both words).
    double *from = A, *to = tmp;
    for (int k = 0, kp = 0, p = 0; kp < n; ++p) {
      const int e = std::min(n, k + kPanel), npan = k < n ? (n + kPanel - 1) / kPanel : 0;
      const size_t lds = mt * nt <= kStepOneTiles ? kStepLdsOne : kStepLdsTwo;
      hipLaunchKernelGGL(gje_block_step_kernel, dim3(npan + mt * nt), dim3(kBpThreads), lds, s, n, npan, kp, k, k, e,
                         from, to, swp + ((p + 1) & 1) * kPanel, swp + (p & 1) * kPanel, piv, status + ((p + 1) & 1),
                         status + (p & 1));
      std::swap(from, to);
      kp = k;
      k = e;
    }
    A = from;
    tmp = to;
  } else if (R > 0) {
    // Elimination of each panel in one cooperative launch with a look-ahead:
    // the update by panel p first brings the next panel's columns up to date,
    // then the next panel is eliminated on s
    // while the rest of the update runs on the side stream.  The two touch
    // different columns, and the next panel's swaps on the other columns wait
    // for the rest of the update.  Every entry gets the same updates as
    // without the look-ahead, bit for bit.
    auto eliminate = [&](int k, int e) {
      int n_ = n, k_ = k, e_ = e, R_ = R;
      GjSync gs_ = gs;
      unsigned bar0 = (unsigned)k;
      void *args[] = {&n_, &k_, &e_, &R_, &A, &piv, &swp, &gs_, &bar0, &status};
      STKKT_HIP(hipLaunchCooperativeKernel(reinterpret_cast<const void *>(&gje_panel_kernel),
                                           dim3((n + R - 1) / R), dim3(kGjThreads), args,
                                           (unsigned)(sizeof(double) * (size_t)kPanel * (R + 1)), s));
    };
    eliminate(0, std::min(n, kPanel));
    close_panel(0, std::min(n, kPanel), rows);
    for (int k = 0, p = 0; k < n; k += kPanel, ++p) {
      const int e = std::min(n, k + kPanel);
      double *Rk = rows + (size_t)(p & 1) * kPanel * n;
      if (e >= n) {
        update(k, e, 0, n, 0, 0, Rk, s);
        break;
      }
      const int e2 = std::min(n, e + kPanel);
      STKKT_HIP(hipEventRecord(la.rows_ready, s));
      update(k, e, e, e2, 0, 0, Rk, s);
      STKKT_HIP(hipStreamWaitEvent(la.side, la.rows_ready, 0));
      update(k, e, 0, n, e, e2, Rk, la.side);
      STKKT_HIP(hipEventRecord(la.rest_done, la.side));
      eliminate(e, e2);
      STKKT_HIP(hipStreamWaitEvent(s, la.rest_done, 0));
      close_panel(e, e2, rows + (size_t)((p + 1) & 1) * kPanel * n);
    }
  } else {
    for (int k = 0; k < n; k += kPanel) {
      const int e = std::min(n, k + kPanel);
      const int nrb = (n + 63) / 64;
      hipLaunchKernelGGL(gje_panel_gather_kernel, dim3(nrb), dim3(256), 0, s, n, k, e - k, A, pan);
      for (int c = k; c < e; ++c) {
        hipLaunchKernelGGL(gje_pivot_kernel, dim3(1), dim3(1024), 0, s, n, k, e, c, pan, piv, swp, prow, fcol,
                           status);
        hipLaunchKernelGGL(gje_elim_kernel, dim3((n + 255) / 256, e - k), dim3(256), 0, s, n, k, c, pan, prow,
                           fcol, status);
      }
      hipLaunchKernelGGL(gje_panel_scatter_kernel, dim3(nrb), dim3(256), 0, s, n, k, e - k, pan, A);
      close_panel(k, e, rows);
      update(k, e, 0, n, 0, 0, rows, s);
    }
  }
  hipLaunchKernelGGL(gje_unpermute_kernel, dim3(blocks_for(n, 256, 64), n), dim3(256), 0, s, n, A, piv, tmp);
  STKKT_HIP(hipGetLastError());
  return tmp;
}

CoarseLU::CoarseLU(const Allocator *al, const kkt_op *cop, int precision, hipStream_t s) : prec_(precision) {
  const OpDev &d = cop->d;
  nb_ = 3 * d.N;
  nlev_ = d.M + 1;
  STKKT_REQUIRE(nb_ <= 65535, "coarse_setup: coarse level too large for the dense block solve");
  const size_t nn = (size_t)nb_ * nb_;
  ld_ = (nb_ + kMrRows - 1) / kMrRows * kMrRows;
  const size_t nld = (size_t)ld_ * nb_;
  const size_t esz = precision == STKKT_F32 ? sizeof(float) : sizeof(double);
  Sinv_ = DevBuf(al, esz * nld * nlev_);
  E_ = DevBuf(al, esz * nld * std::max(nlev_ - 1, 1));
  Lidx_ = DevBuf(al, sizeof(int32_t) * (size_t)nb_ * 81 * nlev_);
  Lval_ = DevBuf(al, sizeof(double) * (size_t)nb_ * 81 * nlev_);
  // block products: workgroups of 64 rows x csplit_ columns, 256 of them where
  // that gives the chip enough workgroups (seven levels, one vector and sixteen,
  // 128 / 256 columns, FP64: nb 1029 120 / 144 and 198 / 220 us, 3000 286 / 316
  // and 464 / 478; five levels of nb 6591 624 / 607 and 929 / 878); longer chunks
  // were slower there (FP32 47 us a block with 10 chunks, 56 us with 3, against 41).
  csplit_ = (long long)(ld_ / kMrRows) * ((nb_ + 2 * kMrBatch - 1) / (2 * kMrBatch)) >= 1024 ? 2 * kMrBatch : kMrBatch;
  const size_t gv = (size_t)nb_ * ((nb_ + kGvCols - 1) / kGvCols), nch = (size_t)((nb_ + csplit_ - 1) / csplit_);
  partial_ = DevBuf(al, sizeof(double) * 2 * std::max(gv, nch * ld_ * kMrRhs / 2));
  mt_ = DevBuf(al, sizeof(double) * 2 * (size_t)kMrRhs * nb_);
  y_ = DevBuf(al, sizeof(double) * (size_t)nlev_ * nb_);
  // setup work buffers (FP64)
  DevBuf S(al, sizeof(double) * nn), Ed(al, sizeof(double) * nn),
      tmp(al, sizeof(double) * nn), rows(al, sizeof(double) * 2 * (size_t)kPanel * nb_), piv(al, sizeof(int32_t) * nb_),
      prow(al, sizeof(double) * kPanel), swp(al, sizeof(int32_t) * 2 * kPanel), pan(al, sizeof(double) * kPanel * nb_),
      fcol(al, sizeof(double) * nb_),
      status(al, 256), ridx(al, sizeof(int32_t) * (size_t)nb_ * 81), rval(al, sizeof(double) * (size_t)nb_ * 81),
      cidx(al, sizeof(int32_t) * (size_t)nb_ * 81), cval(al, sizeof(double) * (size_t)nb_ * 81);
  const int nwg_max = (nb_ + 63) / 64;
  DevBuf candv(al, sizeof(double) * 2 * nwg_max), candi(al, sizeof(int32_t) * 2 * nwg_max),
      candrow(al, sizeof(double) * 2 * (size_t)nwg_max * kPanel), crow(al, sizeof(double) * 2 * kPanel),
      bar(al, 256);
  // STKKT_COARSE_SPIN_LIMIT lowers the barrier's poll bound (a test forces the
  // time-out path with it)
  const char *spin_env = std::getenv("STKKT_COARSE_SPIN_LIMIT");
  const unsigned spin = spin_env ? (unsigned)std::max(0, std::atoi(spin_env)) : kGjSpinLimit;
  const GjSync gs{candv.as<double>(), candi.as<int32_t>(), candrow.as<double>(), crow.as<double>(),
                  bar.as<unsigned>(), reinterpret_cast<int *>(bar.as<unsigned char>() + 128), spin};
  STKKT_HIP(hipMemsetAsync(status.ptr, 0, 2 * sizeof(int), s));
  const int G = blocks_for(27LL * d.N, 128, 4096);
  const dim3 g2(blocks_for(nb_, 256, 64), d.N);
  const LookAhead la;
  for (int k = 0; k < nlev_; ++k) {
    // lower coupling of level k (to level k-1), kept for the application
    int32_t *Lk_idx = Lidx_.as<int32_t>() + (size_t)k * nb_ * 81;
    double *Lk_val = Lval_.as<double>() + (size_t)k * nb_ * 81;
    if (k > 0) hipLaunchKernelGGL(coupling_rows_kernel, dim3(G), dim3(128), 0, s, d, k, -1, Lk_idx, Lk_val);
    // S_k = D_k - L_k E_{k-1}
    fill_zero(S.as<double>(), (long long)nn, s);
    hipLaunchKernelGGL(coupling_rows_kernel, dim3(G), dim3(128), 0, s, d, k, 0, ridx.as<int32_t>(),
                       rval.as<double>());
    hipLaunchKernelGGL(dense_from_rows_kernel, dim3(blocks_for(81LL * nb_, 256, 4096)), dim3(256), 0, s, nb_,
                       ridx.as<int32_t>(), rval.as<double>(), S.as<double>());
    if (k > 0) {
      // the level's couplings once more, in the tables of its D_k (used up by now)
      hipLaunchKernelGGL(coupling_nodes_kernel, dim3(G), dim3(128), 0, s, d, k, -1, ridx.as<int32_t>(),
                         rval.as<double>());
      hipLaunchKernelGGL(schur_update_kernel, dim3((d.N + 127) / 128, (nb_ + kSchurCols - 1) / kSchurCols), dim3(128),
                         0, s, d.N, ridx.as<int32_t>(), rval.as<double>(), Ed.as<double>(), S.as<double>());
    }
    STKKT_HIP(hipGetLastError());
    // S_k^{-1} (column-major S is the row-major transpose: invert it as is)
    const double *Sk = gje_invert(nb_, S.as<double>(), tmp.as<double>(), rows.as<double>(), pan.as<double>(),
                                  fcol.as<double>(), piv.as<int32_t>(), swp.as<int32_t>(), prow.as<double>(), gs,
                                  status.as<int>(), la, s);
    // E_k = S_k^{-1} U_k
    if (k + 1 < nlev_) {
      hipLaunchKernelGGL(coupling_cols_kernel, dim3(G), dim3(128), 0, s, d, k, +1, cidx.as<int32_t>(),
                         cval.as<double>());
      hipLaunchKernelGGL(e_from_cols_kernel, g2, dim3(256), 0, s, nb_, cidx.as<int32_t>(), cval.as<double>(),
                         Sk, Ed.as<double>());
      STKKT_HIP(hipGetLastError());
    }
    // store S_k^{-1} and E_k in the application precision, columns padded to ld_
    const dim3 gp(blocks_for(ld_, 256, 64), nb_);
    if (prec_ == STKKT_F32) {
      hipLaunchKernelGGL(store_padded_kernel<float>, gp, dim3(256), 0, s, nb_, ld_, Sk,
                         Sinv_.as<float>() + (size_t)k * nld);
      if (k + 1 < nlev_)
        hipLaunchKernelGGL(store_padded_kernel<float>, gp, dim3(256), 0, s, nb_, ld_, Ed.as<double>(),
                           E_.as<float>() + (size_t)k * nld);
    } else {
      hipLaunchKernelGGL(store_padded_kernel<double>, gp, dim3(256), 0, s, nb_, ld_, Sk,
                         Sinv_.as<double>() + (size_t)k * nld);
      if (k + 1 < nlev_)
        hipLaunchKernelGGL(store_padded_kernel<double>, gp, dim3(256), 0, s, nb_, ld_, Ed.as<double>(),
                           E_.as<double>() + (size_t)k * nld);
    }
    STKKT_HIP(hipGetLastError());
  }
  int st[2] = {0, 0};
  STKKT_HIP(hipMemcpyAsync(st, status.ptr, 2 * sizeof(int), hipMemcpyDeviceToHost, s));
  STKKT_HIP(hipStreamSynchronize(s));   // the setup buffers are released on return
  if (st[0] == 2) throw Error(STKKT_EHIP, "coarse LU: panel elimination barrier timed out");
  if (st[0] || st[1]) throw Error(STKKT_EBREAKDOWN, "coarse LU: singular Schur complement block");
}

// partial = chunk sums of A times the input, q right-hand sides (one on the GEMV when `gemv`)
template <typename T>
void CoarseLU::product(bool gemv, int q, const T *A, const ProductInput &in, double *partial, hipStream_t s) const {
  if constexpr (sizeof(T) == 4) {
    if (gemv) {
      const dim3 grid(ld_ / kGvRows, (nb_ + kGvCols - 1) / kGvCols);
      const auto kernel = nb_ <= fold_rows(true) ? gemv_partial_kernel<64> : gemv_partial_kernel<32>;
      hipLaunchKernelGGL(kernel, grid, dim3(kGvRows), 0, s, nb_, ld_, A, in, partial);
      return;
    }
  }
  const dim3 grid(ld_ / kMrRows, (nb_ + csplit_ - 1) / csplit_);
  const bool one = csplit_ == kMrBatch, sums = q == 1 && nb_ <= fold_rows(false);
  const auto kernel = sums ? (one ? gemm_partial_kernel<T, 1, true> : gemm_partial_kernel<T, 2, true>)
                           : (one ? gemm_partial_kernel<T, 1, false> : gemm_partial_kernel<T, 2, false>);
  hipLaunchKernelGGL(kernel, grid, dim3(kMrThreads), 0, s, nb_, ld_, A, q, in, partial);
}

// The two sweeps for one right-hand side and blocks of at most fold_rows() rows:
// forward, per level, lower_rhs_kernel (t = r_k - L_k y_{k-1}, y_{k-1} from the
// chunk sums of the previous product) and the product by S_k^{-1}; backward one
// launch per level, the product by E_k, whose input x_{k+1} = y_{k+1} - E_{k+1}
// x_{k+2} its workgroups form from the previous product's chunk sums.
template <typename T> void CoarseLU::sweep_one(bool gemv, const double *r, double *x, hipStream_t s) const {
  const size_t nn = (size_t)ld_ * nb_;
  const T *Si = static_cast<const T *>(Sinv_.ptr);
  const T *E = static_cast<const T *>(E_.ptr);
  double *t = mt_.as<double>(), *y = y_.as<double>();
  double *part[2] = {partial_.as<double>(), partial_.as<double>() + partial_.bytes / sizeof(double) / 2};
  ProductInput in{};
  in.nch = gemv ? (nb_ + kGvCols - 1) / kGvCols : (nb_ + csplit_ - 1) / csplit_;
  in.ld = gemv ? nb_ : ld_;
  int cur = 0;   // part[cur]: the last product
  for (int k = 0; k < nlev_; ++k) {
    hipLaunchKernelGGL(lower_rhs_kernel, dim3(blocks_for(nb_, 4, 1 << 16)), dim3(256), 0, s, nb_, in.ld, in.nch,
                       Lidx_.as<int32_t>() + (size_t)k * nb_ * 81, Lval_.as<double>() + (size_t)k * nb_ * 81,
                       r + (size_t)k * nb_, k > 0 ? part[cur] : nullptr, k > 0 ? y + (size_t)(k - 1) * nb_ : nullptr, t,
                       1);
    in.vec = t;
    in.vsi = 1;
    product(gemv, 1, Si + (size_t)k * nn, in, part[cur ^ 1], s);
    cur ^= 1;
  }
  // x_M = y_M: the chunk sums of the last product; then x_k = y_k - E_k x_{k+1}
  in.vec = nullptr;
  for (int k = nlev_ - 1; k >= 0; --k) {
    in.partial = part[cur];
    in.base = k + 1 < nlev_ ? y + (size_t)k * nb_ : nullptr;
    in.out = x + (size_t)k * nb_;
    if (k == 0) {
      hipLaunchKernelGGL(product_finish_kernel, dim3(blocks_for(nb_, 64, 4096)), dim3(64), 0, s, nb_, in);
      break;
    }
    product(gemv, 1, E + (size_t)(k - 1) * nn, in, part[cur ^ 1], s);   // writes x_k on the way
    cur ^= 1;
  }
  STKKT_HIP(hipGetLastError());
}

// The same for q <= 16 right-hand sides (one on the GEMV when `gemv`), the
// chunk sums added by a launch of their own that also leaves the next product's
// input transposed.
template <typename T>
void CoarseLU::sweep_multi(bool gemv, int q, const double *r, long long ldr, double *x, long long ldx,
                           hipStream_t s) const {
  const size_t nn = (size_t)ld_ * nb_;
  const T *Si = static_cast<const T *>(Sinv_.ptr);
  const T *E = static_cast<const T *>(E_.ptr);
  double *t = mt_.as<double>(), *xT = t + (size_t)kMrRhs * nb_, *part = partial_.as<double>();
  const int nch = gemv ? (nb_ + kGvCols - 1) / kGvCols : (nb_ + csplit_ - 1) / csplit_, ldp = gemv ? nb_ : ld_;
  ProductInput in{};
  in.vsi = q;
  auto reduce = [&](const double *base, double *out) {
    hipLaunchKernelGGL(gemm_reduce_kernel, dim3(blocks_for(nb_, 64, 4096), q), dim3(64), 0, s, nb_, ldp, q, nch, part,
                       base, ldx, out, ldx, xT, q);
  };
  const int vecs = q == 1 ? 1 : q == 2 ? 2 : 4;
  const auto lower_rhs = vecs == 1   ? lower_rhs_multi_kernel<1>
                         : vecs == 2 ? lower_rhs_multi_kernel<2>
                                     : lower_rhs_multi_kernel<4>;
  // forward: y_k kept in x (the last one also in xT)
  for (int k = 0; k < nlev_; ++k) {
    hipLaunchKernelGGL(lower_rhs, dim3(blocks_for(nb_, 4, 1 << 16), (q + vecs - 1) / vecs), dim3(256), 0, s, nb_, q,
                       Lidx_.as<int32_t>() + (size_t)k * nb_ * 81, Lval_.as<double>() + (size_t)k * nb_ * 81,
                       r + (size_t)k * nb_, ldr, k > 0 ? x + (size_t)(k - 1) * nb_ : nullptr, ldx, t, q);
    in.vec = t;
    product(gemv, q, Si + (size_t)k * nn, in, part, s);
    reduce(nullptr, x + (size_t)k * nb_);
  }
  in.vec = xT;
  for (int k = nlev_ - 2; k >= 0; --k) {
    product(gemv, q, E + (size_t)k * nn, in, part, s);
    reduce(x + (size_t)k * nb_, x + (size_t)k * nb_);
  }
  STKKT_HIP(hipGetLastError());
}

template <typename T> void CoarseLU::solve_one(bool gemv, const double *r, double *x, hipStream_t s) const {
  if (nb_ <= fold_rows(gemv)) sweep_one<T>(gemv, r, x, s);
  else sweep_multi<T>(gemv, 1, r, 0, x, 0, s);
}

void CoarseLU::solve(const double *r, double *x, hipStream_t s) const {
  if (prec_ == STKKT_F32) solve_one<float>(true, r, x, s);
  else solve_one<double>(false, r, x, s);
}

void CoarseLU::solve_multi(int q, const double *r, long long ldr, double *x, long long ldx, hipStream_t s) const {
  for (int c0 = 0; c0 < q; c0 += kMrRhs) {
    const int qq = std::min(kMrRhs, q - c0);
    const double *rg = r + c0 * ldr;
    double *xg = x + c0 * ldx;
    if (prec_ == STKKT_F32) {
      if (qq == 1) solve_one<float>(false, rg, xg, s);
      else sweep_multi<float>(false, qq, rg, ldr, xg, ldx, s);
    } else {
      if (qq == 1) solve_one<double>(false, rg, xg, s);
      else sweep_multi<double>(false, qq, rg, ldr, xg, ldx, s);
    }
  }
}

size_t CoarseLU::bytes_per_solve() const {
  const size_t esz = prec_ == STKKT_F32 ? sizeof(float) : sizeof(double);
  return esz * (size_t)nb_ * nb_ * (2 * nlev_ - 1);
}

}  // namespace stkkt
