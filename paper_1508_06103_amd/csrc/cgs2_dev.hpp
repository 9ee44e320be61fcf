// Device bodies of the fused classical Gram-Schmidt passes, shared by the
// single-solve kernels and the batched ones: each workgroup of 256 threads
// (four wavefronts) takes one element range [lo, hi) and leaves per-range
// partial sums that a second stage adds in a fixed order.
#pragma once

#include <type_traits>

#include "common.hpp"

namespace stkkt {

constexpr int kCgsThreads = 256;
constexpr int kCgsMaxK = 64;   // basis vectors a fused pass accepts

// f(width) with the smallest multiple of eight >= k (1 <= k <= kCgsMaxK) as a
// compile-time width: the passes below keep one register per basis vector.
template <typename F> inline void with_cgs_width(int k, F f) {
  switch ((k + 7) / 8) {
    case 0:
    case 1: return f(std::integral_constant<int, 8>{});
    case 2: return f(std::integral_constant<int, 16>{});
    case 3: return f(std::integral_constant<int, 24>{});
    case 4: return f(std::integral_constant<int, 32>{});
    case 5: return f(std::integral_constant<int, 40>{});
    case 6: return f(std::integral_constant<int, 48>{});
    case 7: return f(std::integral_constant<int, 56>{});
    default: return f(std::integral_constant<int, 64>{});
  }
}

// Entries e of the basis vectors 0 .. k - 1 into v[0 .. KR), zeros past k or
// for an invalid element.  The loads carry no branch (a vector past k reads the
// last one's entry, an invalid element the caller's in-range `e`), so that all
// of them are in flight together.
template <int KR>
__device__ inline void load_basis(const double *__restrict__ V, long long ldv, int k, long long e, bool valid,
                                  double (&v)[KR]) {
  double x[KR];
#pragma unroll
  for (int j = 0; j < KR; ++j) x[j] = V[(long long)min(j, k - 1) * ldv + e];
#pragma unroll
  for (int j = 0; j < KR; ++j) v[j] = j < k && valid ? x[j] : 0.0;
}

__device__ inline double cgs_wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

// Tiles of one wavefront: lanes are elements, a wavefront takes 64-element
// tiles; the KR >= k basis entries of a tile are loaded once into registers
// and serve both the update and the dots, so V is read once.  The
// wavefront's dot sums go to red[wave][g].
template <int KR>
__device__ inline void update_dot_tiles(double *__restrict__ w, const double *__restrict__ V, long long ldv, int k,
                                        cptr<double> hc, long long lo, long long hi,
                                        double (*red)[kCgsMaxK]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long ntiles = (hi - lo + 63) / 64;
  double acc[KR];
#pragma unroll
  for (int j = 0; j < KR; ++j) acc[j] = 0.0;
  for (long long t = wave; t < ntiles; t += kCgsThreads / 64) {
    const long long e = lo + 64 * t + lane;
    const bool valid = e < hi;
    const long long ec = valid ? e : hi - 1;
    const double wold = w[ec];
    double v[KR];
    load_basis<KR>(V, ldv, k, ec, valid, v);
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < KR; ++j) s = __builtin_fma(j < k ? hc[j] : 0.0, v[j], s);
    const double wn = valid ? wold - s : 0.0;
    if (valid) w[e] = wn;
#pragma unroll
    for (int j = 0; j < KR; ++j) acc[j] = __builtin_fma(v[j], wn, acc[j]);
  }
#pragma unroll
  for (int j = 0; j < KR; ++j)
    if (j < k) {
      const double r = cgs_wave_sum(acc[j]);
      if (lane == 0) red[wave][j] = r;
    }
}

// out[g * ostride] = sum over [lo, hi) of V_g[e] w[e], g < k <= KR: the same
// tiles as the update+dot, without the update (the first CGS pass).
template <int KR>
__device__ inline void dot_range(const double *__restrict__ w, const double *__restrict__ V, long long ldv, int k,
                                 long long lo, long long hi, double *__restrict__ out, long long ostride) {
  __shared__ double red[kCgsThreads / 64][kCgsMaxK];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long ntiles = (hi - lo + 63) / 64;
  double acc[KR];
#pragma unroll
  for (int j = 0; j < KR; ++j) acc[j] = 0.0;
  for (long long t = wave; t < ntiles; t += kCgsThreads / 64) {
    const long long e = lo + 64 * t + lane;
    const bool valid = e < hi;
    const long long ec = valid ? e : hi - 1;
    const double wold = w[ec], we = valid ? wold : 0.0;
    double v[KR];
    load_basis<KR>(V, ldv, k, ec, valid, v);
#pragma unroll
    for (int j = 0; j < KR; ++j) acc[j] = __builtin_fma(v[j], we, acc[j]);
  }
#pragma unroll
  for (int j = 0; j < KR; ++j)
    if (j < k) {
      const double r = cgs_wave_sum(acc[j]);
      if (lane == 0) red[wave][j] = r;
    }
  __syncthreads();
  if ((int)threadIdx.x < k) {
    double s = 0.0;
#pragma unroll
    for (int wv = 0; wv < kCgsThreads / 64; ++wv) s += red[wv][threadIdx.x];
    out[(long long)threadIdx.x * ostride] = s;
  }
}

// w[e] <- w[e] - sum_{g<k} h[g] V_g[e] for e in [lo, hi), then
// out[g * ostride] = sum over the range of V_g[e] w_new[e], g < k <= KR.
// Every wavefront works on its own tiles with no synchronisation.  KR is the
// smallest multiple of eight >= k: more registers per wavefront, fewer
// wavefronts per SIMD, more loads in flight per wavefront.
template <int KR>
__device__ inline void update_dot_range(double *__restrict__ w, const double *__restrict__ V, long long ldv, int k,
                                        const double *__restrict__ h, long long lo, long long hi,
                                        double *__restrict__ out, long long ostride) {
  __shared__ double red[kCgsThreads / 64][kCgsMaxK];
  update_dot_tiles<KR>(w, V, ldv, k, as_const(h), lo, hi, red);
  __syncthreads();
  if ((int)threadIdx.x < k) {
    double s = 0.0;
#pragma unroll
    for (int wv = 0; wv < kCgsThreads / 64; ++wv) s += red[wv][threadIdx.x];
    out[(long long)threadIdx.x * ostride] = s;
  }
}

// w[e] <- w[e] - sum_{g<k} h[g] V_g[e] for e in [lo, hi); returns (in thread
// 0) the range's sum of w_new[e]^2.
// The basis entries of an element are loaded together (up to KR, KR >= k;
// instantiated like the update+dot) before the sum, in the same order.
template <int KR>
__device__ inline double update_norm_range(double *__restrict__ w, const double *__restrict__ V, long long ldv, int k,
                                           const double *__restrict__ h, long long lo, long long hi) {
  __shared__ double red[kCgsThreads / 64];
  const cptr<double> hc = as_const(h);
  double acc = 0.0;
  for (long long e = lo + threadIdx.x; e < hi; e += kCgsThreads) {
    const double wold = w[e];
    double v[KR];
    load_basis<KR>(V, ldv, k, e, true, v);
    double s = 0.0;
#pragma unroll
    for (int g = 0; g < KR; ++g) s = __builtin_fma(g < k ? hc[g] : 0.0, v[g], s);
    const double wn = wold - s;
    w[e] = wn;
    acc = __builtin_fma(wn, wn, acc);
  }
  acc = cgs_wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int wv = 0; wv < kCgsThreads / 64; ++wv) s += red[wv];
  return s;
}

}  // namespace stkkt
