// FP64 vector kernels for the Krylov solvers: fixed-order two-stage
// reductions (reproducible run to run) built on wavefront shuffles, and the
// streaming updates of classical Gram-Schmidt.
#include "common.hpp"
#include "krylov.hpp"
#include "cgs2_dev.hpp"

namespace stkkt {

namespace {

constexpr int kThreads = 256;
constexpr int kGroup = 8;   // vectors per pass of the multi-dot

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

// partial[i * G + b] = sum over block b's elements of V_i[e] * w[e], i < k.
__global__ void __launch_bounds__(kThreads) multidot_kernel(const double *__restrict__ V, long long ldv, int k,
                                                            const double *__restrict__ w, long long n,
                                                            double *__restrict__ partial) {
  __shared__ double red[kGroup][kThreads / 64];
  const int G = gridDim.x;
  const long long per = (n + G - 1) / G;
  const long long lo = (long long)blockIdx.x * per;
  const long long hi = lo + per < n ? lo + per : n;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int i0 = 0; i0 < k; i0 += kGroup) {
    const int gk = k - i0 < kGroup ? k - i0 : kGroup;
    double acc[kGroup];
#pragma unroll
    for (int g = 0; g < kGroup; ++g) acc[g] = 0.0;
    for (long long e = lo + threadIdx.x; e < hi; e += kThreads) {
      const double we = w[e];
#pragma unroll
      for (int g = 0; g < kGroup; ++g)
        if (g < gk) acc[g] += V[(long long)(i0 + g) * ldv + e] * we;
    }
#pragma unroll
    for (int g = 0; g < kGroup; ++g) {
      const double s = wave_sum(acc[g]);
      if (lane == 0) red[g][wave] = s;
    }
    __syncthreads();
    if ((int)threadIdx.x < gk) {
      double s = 0.0;
      for (int wv = 0; wv < kThreads / 64; ++wv) s += red[threadIdx.x][wv];
      partial[(long long)(i0 + threadIdx.x) * G + blockIdx.x] = s;
    }
    __syncthreads();
  }
}

// The first CGS pass for k <= 64 vectors on the register tiles of the fused
// passes (partial[i * G + b] as above).
template <int KR>
__global__ void __launch_bounds__(kCgsThreads) multidot_tiles_kernel(const double *__restrict__ V, long long ldv,
                                                                     int k, const double *__restrict__ w, long long n,
                                                                     double *__restrict__ partial) {
  const int G = gridDim.x;
  const long long per = (n + G - 1) / G;
  const long long lo = (long long)blockIdx.x * per;
  const long long hi = lo + per < n ? lo + per : n;
  dot_range<KR>(w, V, ldv, k, lo, hi > lo ? hi : lo, partial + blockIdx.x, G);
}

// out[i] = sum_b partial[i * G + b] (fixed order), one block per i.
__global__ void __launch_bounds__(kThreads) reduce_kernel(const double *__restrict__ partial, int G,
                                                          double *__restrict__ out) {
  __shared__ double red[kThreads / 64];
  const int i = blockIdx.x;
  double s = 0.0;
  for (int b = threadIdx.x; b < G; b += kThreads) s += partial[(long long)i * G + b];
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int wv = 0; wv < kThreads / 64; ++wv) t += red[wv];
    out[i] = t;
  }
}

// w[e] -= sum_i h[i] V_i[e]   (h in device memory, i ascending)
__global__ void __launch_bounds__(kThreads) update_kernel(double *__restrict__ w, const double *__restrict__ V,
                                                          long long ldv, int k, const double *__restrict__ h,
                                                          long long n) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
    double s = 0.0;
    for (int i = 0; i < k; ++i) s += h[i] * V[(long long)i * ldv + e];
    w[e] -= s;
  }
}

// out[e] = sum_i y[i] V_i[e]  (+ out[e] if accumulate)
__global__ void __launch_bounds__(kThreads) combine_kernel(double *__restrict__ out, const double *__restrict__ V,
                                                           long long ldv, int k, const double *__restrict__ y,
                                                           long long n, int accumulate) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
    double s = 0.0;
    for (int i = 0; i < k; ++i) s += y[i] * V[(long long)i * ldv + e];
    out[e] = accumulate ? out[e] + s : s;
  }
}

// out = a * x + b * y
__global__ void __launch_bounds__(kThreads) axpby_kernel(double *__restrict__ out, double a, const double *__restrict__ x,
                                                         double b, const double *__restrict__ y, long long n) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x)
    out[e] = a * x[e] + b * y[e];
}

__global__ void scale_kernel(double *__restrict__ out, const double *__restrict__ x, double a, long long n) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x)
    out[e] = a * x[e];
}

// Second CGS pass fused with the first update (w <- w - V h, partial[g * G +
// b] = block b's part of V_g . w_new) and the last update fused with the norm
// (partial[b] = block b's part of |w_new|^2); the bodies are shared with the
// batched solver.
template <int KR>
__global__ void __launch_bounds__(kCgsThreads) update_dot_kernel(double *__restrict__ w, const double *__restrict__ V,
                                                                 long long ldv, int k, const double *__restrict__ h,
                                                                 long long n, double *__restrict__ partial) {
  const int G = gridDim.x;
  const long long per = (n + G - 1) / G;
  const long long lo = (long long)blockIdx.x * per;
  const long long hi = lo + per < n ? lo + per : n;
  update_dot_range<KR>(w, V, ldv, k, h, lo, hi > lo ? hi : lo, partial + blockIdx.x, G);
}

template <int KR>
__global__ void __launch_bounds__(kCgsThreads) update_norm_kernel(double *__restrict__ w, const double *__restrict__ V,
                                                                  long long ldv, int k, const double *__restrict__ h,
                                                                  long long n, double *__restrict__ partial) {
  const int G = gridDim.x;
  const long long per = (n + G - 1) / G;
  const long long lo = (long long)blockIdx.x * per;
  const long long hi = lo + per < n ? lo + per : n;
  const double s = update_norm_range<KR>(w, V, ldv, k, h, lo, hi > lo ? hi : lo);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// Short vectors: at most kSmallRanges ranges of up to 4096 elements leave most
// of the chip idle in the kernels above, each workgroup reading its tiles one
// after the other.  The update then runs on its own over all elements and the
// dots take kSmallDots vectors per workgroup with all of a wavefront's tiles
// in flight; every sum is the one of the kernels above, in the same order and
// with the same fused multiply-adds, so both forms give the same bits.  At
// n = 37 000 and 18 vectors the three passes of a step took 21, 33 and 33 us
// on 10 workgroups, now 6, 5 + 6 and 5 + 5.  The limit is one range per compute
// unit: 30 steps at n = 165 000 (41 ranges) 16.0 -> 14.6 ms, 695 000 (170) 30.0
// -> 29.7, 1 172 000 (287) no difference, 2 297 000 (561) slower by the second
// read of V.
constexpr int kSmallRanges = 256, kSmallDots = 4, kSmallTiles = 4096 / 64 / (kCgsThreads / 64);

__global__ void __launch_bounds__(kCgsThreads) small_dots_kernel(const double *__restrict__ V, long long ldv, int k,
                                                                 const double *__restrict__ w, long long n,
                                                                 double *__restrict__ partial) {
  __shared__ double red[kCgsThreads / 64][kSmallDots];
  const int G = gridDim.x, j0 = blockIdx.y * kSmallDots;
  const long long per = (n + G - 1) / G, lo = (long long)blockIdx.x * per, hi = lo + per < n ? lo + per : n;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double v[kSmallTiles][kSmallDots], we[kSmallTiles];
#pragma unroll
  for (int i = 0; i < kSmallTiles; ++i) {
    const long long e = lo + 64 * (wave + (kCgsThreads / 64) * i) + lane;
    const long long ec = e < hi ? e : n - 1;
    we[i] = w[ec];
#pragma unroll
    for (int j = 0; j < kSmallDots; ++j) v[i][j] = V[(long long)min(j0 + j, k - 1) * ldv + ec];
  }
  double acc[kSmallDots];
#pragma unroll
  for (int j = 0; j < kSmallDots; ++j) acc[j] = 0.0;
#pragma unroll
  for (int i = 0; i < kSmallTiles; ++i) {
    const bool valid = lo + 64 * (wave + (kCgsThreads / 64) * i) + lane < hi;
#pragma unroll
    for (int j = 0; j < kSmallDots; ++j) acc[j] = valid ? __builtin_fma(v[i][j], we[i], acc[j]) : acc[j];
  }
#pragma unroll
  for (int j = 0; j < kSmallDots; ++j) {
    const double r = cgs_wave_sum(acc[j]);
    if (lane == 0) red[wave][j] = r;
  }
  __syncthreads();
  const int j = (int)threadIdx.x;
  if (j < kSmallDots && j0 + j < k) {
    double s = 0.0;
#pragma unroll
    for (int wv = 0; wv < kCgsThreads / 64; ++wv) s += red[wv][j];
    partial[(long long)(j0 + j) * G + blockIdx.x] = s;
  }
}

template <int KR>
__global__ void __launch_bounds__(kCgsThreads) small_update_kernel(double *__restrict__ w, const double *__restrict__ V,
                                                                   long long ldv, int k, const double *__restrict__ h,
                                                                   long long n) {
  const long long e = blockIdx.x * (long long)kCgsThreads + threadIdx.x;
  const bool valid = e < n;
  const cptr<double> hc = as_const(h);
  const double wold = w[valid ? e : n - 1];
  double v[KR];
  load_basis<KR>(V, ldv, k, valid ? e : n - 1, true, v);
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < KR; ++j) s = __builtin_fma(j < k ? hc[j] : 0.0, v[j], s);
  if (valid) w[e] = wold - s;
}

__global__ void __launch_bounds__(kCgsThreads) small_norm_kernel(const double *__restrict__ w, long long n,
                                                                 double *__restrict__ partial) {
  __shared__ double red[kCgsThreads / 64];
  const int G = gridDim.x;
  const long long per = (n + G - 1) / G, lo = (long long)blockIdx.x * per, hi = lo + per < n ? lo + per : n;
  double v[4096 / kCgsThreads];
#pragma unroll
  for (int i = 0; i < 4096 / kCgsThreads; ++i) {
    const long long e = lo + threadIdx.x + (long long)kCgsThreads * i;
    v[i] = w[e < hi ? e : n - 1];
    v[i] = e < hi ? v[i] : 0.0;
  }
  double acc = 0.0;
#pragma unroll
  for (int i = 0; i < 4096 / kCgsThreads; ++i) acc = __builtin_fma(v[i], v[i], acc);
  acc = cgs_wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int wv = 0; wv < kCgsThreads / 64; ++wv) s += red[wv];
    partial[blockIdx.x] = s;
  }
}

void launch_small_dots(const double *w, const double *V, long long ldv, int k, long long n, int G, double *partial,
                       hipStream_t s) {
  hipLaunchKernelGGL(small_dots_kernel, dim3(G, (k + kSmallDots - 1) / kSmallDots), dim3(kCgsThreads), 0, s, V, ldv, k,
                     w, n, partial);
}

void launch_update(double *w, const double *V, long long ldv, int k, const double *h, long long n, hipStream_t s) {
  with_cgs_width(k, [&](auto width) {
    hipLaunchKernelGGL(small_update_kernel<decltype(width)::value>, dim3((unsigned)((n + kCgsThreads - 1) / kCgsThreads)),
                       dim3(kCgsThreads), 0, s, w, V, ldv, k, h, n);
  });
}

}  // namespace

bool cgs2_fused_ok(int k) { return k <= kCgsMaxK; }

void update_dot(double *w, const double *V, long long ldv, int k, const double *h, long long n, double *partial,
                double *out, hipStream_t s) {
  const int G = reduction_blocks(n);
  if (G <= kSmallRanges) {
    launch_update(w, V, ldv, k, h, n, s);
    launch_small_dots(w, V, ldv, k, n, G, partial, s);
  } else {
    with_cgs_width(k, [&](auto width) {
      hipLaunchKernelGGL(update_dot_kernel<decltype(width)::value>, dim3(G), dim3(kCgsThreads), 0, s, w, V, ldv, k, h,
                         n, partial);
    });
  }
  STKKT_HIP(hipGetLastError());
  hipLaunchKernelGGL(reduce_kernel, dim3(k), dim3(kThreads), 0, s, partial, G, out);
  STKKT_HIP(hipGetLastError());
}

void update_norm(double *w, const double *V, long long ldv, int k, const double *h, long long n, double *partial,
                 double *out, hipStream_t s) {
  const int G = reduction_blocks(n);
  if (G <= kSmallRanges) {
    launch_update(w, V, ldv, k, h, n, s);
    hipLaunchKernelGGL(small_norm_kernel, dim3(G), dim3(kCgsThreads), 0, s, w, n, partial);
  } else {
    with_cgs_width(k, [&](auto width) {
      hipLaunchKernelGGL(update_norm_kernel<decltype(width)::value>, dim3(G), dim3(kCgsThreads), 0, s, w, V, ldv, k, h,
                         n, partial);
    });
  }
  STKKT_HIP(hipGetLastError());
  hipLaunchKernelGGL(reduce_kernel, dim3(1), dim3(kThreads), 0, s, partial, G, out);
  STKKT_HIP(hipGetLastError());
}

int reduction_blocks(long long n) {
  long long g = (n + 4095) / 4096;
  if (g > 2048) g = 2048;
  if (g < 1) g = 1;
  return (int)g;
}

void multidot(const double *V, long long ldv, int k, const double *w, long long n, double *partial, double *out,
              hipStream_t s) {
  const int G = reduction_blocks(n);
  if (G <= kSmallRanges)
    launch_small_dots(w, V, ldv, k, n, G, partial, s);
  else if (k <= kCgsMaxK)
    with_cgs_width(k, [&](auto width) {
      hipLaunchKernelGGL(multidot_tiles_kernel<decltype(width)::value>, dim3(G), dim3(kCgsThreads), 0, s, V, ldv, k, w,
                         n, partial);
    });
  else
    hipLaunchKernelGGL(multidot_kernel, dim3(G), dim3(kThreads), 0, s, V, ldv, k, w, n, partial);
  STKKT_HIP(hipGetLastError());
  hipLaunchKernelGGL(reduce_kernel, dim3(k), dim3(kThreads), 0, s, partial, G, out);
  STKKT_HIP(hipGetLastError());
}

void gs_update(double *w, const double *V, long long ldv, int k, const double *h, long long n, hipStream_t s) {
  hipLaunchKernelGGL(update_kernel, dim3(blocks_for(n, kThreads, 16384)), dim3(kThreads), 0, s, w, V, ldv, k, h, n);
  STKKT_HIP(hipGetLastError());
}

void combine(double *out, const double *V, long long ldv, int k, const double *y, long long n, bool accumulate,
             hipStream_t s) {
  hipLaunchKernelGGL(combine_kernel, dim3(blocks_for(n, kThreads, 16384)), dim3(kThreads), 0, s, out, V, ldv, k, y,
                     n, accumulate ? 1 : 0);
  STKKT_HIP(hipGetLastError());
}

void axpby(double *out, double a, const double *x, double b, const double *y, long long n, hipStream_t s) {
  hipLaunchKernelGGL(axpby_kernel, dim3(blocks_for(n, kThreads, 16384)), dim3(kThreads), 0, s, out, a, x, b, y, n);
  STKKT_HIP(hipGetLastError());
}

void scale(double *out, const double *x, double a, long long n, hipStream_t s) {
  hipLaunchKernelGGL(scale_kernel, dim3(blocks_for(n, kThreads, 16384)), dim3(kThreads), 0, s, out, x, a, n);
  STKKT_HIP(hipGetLastError());
}

}  // namespace stkkt
