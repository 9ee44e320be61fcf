// Two-level space-time preconditioner (Section 3.2, two-level paragraph):
// nested coarse space-time mesh, linear interpolation I_c^h and its transpose
// (or injection) as transfers, and the coarse KKT system rediscretised on the
// coarse mesh.  F_c^{-1} is applied either as in the paper's experiments
// (Section 4): a few steps of restarted GMRES from zero, right-preconditioned
// by the one-level space-time RAS of the coarse mesh; or exactly, by block
// elimination in time with explicitly inverted Schur complements (CoarseLU).
#include <algorithm>
#include <cmath>
#include <memory>
#include <vector>

#include "coarse.hpp"
#include "coarse_lu.hpp"
#include "ras.hpp"

struct coarse {
  stkkt::Allocator al;
  const kkt_op *fine_op = nullptr;   // identity only
  stkkt::OpDev fine{};
  int fac[4] = {1, 1, 1, 1};
  coarse_params_t params{};
  kkt_op *cop = nullptr;    // owned coarse operator
  ras *cras = nullptr;      // owned coarse preconditioner
  stkkt::DevBuf xc, yc;     // coarse vectors
  stkkt::DevBuf rt[2];      // intermediate vectors of the axis-by-axis restriction
  // coarse vectors of several right-hand sides (exact coarse solve), grown on demand
  mutable stkkt::DevBuf xcm, ycm, midm;
  mutable int mcap = 0;
  std::unique_ptr<stkkt::GmresWork> work;   // inner GMRES workspace
  std::unique_ptr<stkkt::CoarseLU> lu;       // exact coarse solve (method LU)
  ~coarse() {
    lu.reset();
    work.reset();
    delete cras;
    delete cop;
  }
};

namespace stkkt {

namespace {

// 1-D linear interpolation weight of coarse node I at fine node i (factor f,
// rf = 1 / f): (f - |i - I f|) / f inside the support, else 0.
__device__ inline double hat(int i, int I, int f, double rf) {
  const int d = i - I * f;
  const int ad = d < 0 ? -d : d;
  return ad >= f ? 0.0 : (double)(f - ad) * rf;
}

// Vectors of one launch of a transfer (blockIdx.y selects one).
constexpr int kTransferVecs = 4;
struct VecsIn {
  const double *p[kTransferVecs];
};
struct VecsOut {
  double *p[kTransferVecs];
};

// y_fine = I_c^h x_coarse: every fine node interpolates the (up to 16) coarse
// nodes of the coarse space-time cell that contains it (the interpolation is
// the tensor product of the 1-D hat functions).  A thread owns one entry (x
// node and component) of the fine lines of one coarse (y, z) cell group at one
// time level, i1 in [g1 fy, g1 fy + fy), i2 in [g2 fz, g2 fz + fz) (the last
// group of an axis is its last node alone): it blends the four coarse lines at
// its x position in time and x, 16 loads from the coarse vector in L2, and
// writes its fy fz fine values, each a bilinear blend of the four; consecutive
// threads write consecutive entries of a line.  Bound by the fine vector
// written: 56 MB of a 32^3 x 64 mesh in 16 us, 27 us with the lines staged in
// LDS (tables and three barriers per 12 KB of output).
__global__ void __launch_bounds__(256) prolong_kernel(OpDev fo, OpDev co, int fx, int fy, int fz, int ft, VecsIn xs,
                                                      VecsOut ys) {
  const int gy = (fo.nn[1] - 1) / fy + 1, gz = (fo.nn[2] - 1) / fz + 1, len = 3 * fo.nn[0], clen = 3 * co.nn[0];
  const long long total = (long long)len * gy * gz * (fo.M + 1);
  const double *__restrict__ xc = xs.p[blockIdx.y];
  double *__restrict__ y = ys.p[blockIdx.y];
  const double ry = 1.0 / fy, rz = 1.0 / fz;
  for (long long q = blockIdx.x * (long long)blockDim.x + threadIdx.x; q < total;
       q += (long long)gridDim.x * blockDim.x) {
    const long long grp = q / len;
    const int t = (int)(q - grp * len);
    const int g1 = (int)(grp % gy), g2 = (int)((grp / gy) % gz), n = (int)(grp / ((long long)gy * gz));
    const int i0 = t / 3, lo0 = i0 / fx, u0 = 3 * lo0 + (t - 3 * i0), lo3 = n / ft;
    const double wx0 = hat(i0, lo0, fx, 1.0 / fx), wx1 = 1.0 - wx0, wt0 = hat(n, lo3, ft, 1.0 / ft), wt1 = 1.0 - wt0;
    const int ly = min(fy, fo.nn[1] - g1 * fy), lz = min(fz, fo.nn[2] - g2 * fz);
    // steps to the upper coarse neighbours (0 where the node sits on a coarse one: not used then)
    const int sx = i0 % fx != 0 ? 3 : 0, sy = ly > 1 ? clen : 0;
    const long long sz = lz > 1 ? (long long)co.nn[1] * clen : 0, st = n % ft != 0 ? 3LL * co.N : 0;
    const double *c = xc + 3LL * lo3 * co.N + ((long long)co.nn[1] * g2 + g1) * clen + u0;
    double W[2][2];   // [z][y]
#pragma unroll
    for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
      for (int b1 = 0; b1 < 2; ++b1) {
        const double *p = c + b1 * sy + b2 * sz;
        double v = wx0 * p[0];
        if (sx) v += wx1 * p[sx];
        v *= wt0;
        if (st) {
          double w = wx0 * p[st];
          if (sx) w += wx1 * p[st + sx];
          v += wt1 * w;
        }
        W[b2][b1] = v;
      }
    double *o = y + (((long long)n * fo.nn[2] + g2 * fz) * fo.nn[1] + g1 * fy) * len + t;
    for (int jz = 0; jz < lz; ++jz) {
      const double wz0 = (double)(fz - jz) * rz, wz1 = (double)jz * rz;
      double a = wz0 * W[0][0], b = wz0 * W[0][1];
      if (jz > 0) {
        a += wz1 * W[1][0];
        b += wz1 * W[1][1];
      }
      double *ol = o + (long long)jz * fo.nn[1] * len;
      ol[0] = a;
      for (int jy = 1; jy < ly; ++jy) ol[(long long)jy * len] = (double)(fy - jy) * ry * a + (double)jy * ry * b;
    }
  }
}

// x_coarse = injection of x_fine (the fine value at every coarse node)
__global__ void inject_kernel(OpDev fo, OpDev co, int fx, int fy, int fz, int ft, const double *__restrict__ x,
                              double *__restrict__ xc) {
  for (long long g = blockIdx.x * (long long)blockDim.x + threadIdx.x; g < co.V;
       g += (long long)gridDim.x * blockDim.x) {
    const int n = (int)(g / co.N);
    const long long j = g - (long long)n * co.N;
    const int I0 = (int)(j % co.nn[0]), I1 = (int)((j / co.nn[0]) % co.nn[1]),
              I2 = (int)(j / ((long long)co.nn[0] * co.nn[1]));
    const long long fg =
        3 * ((long long)(n * ft) * fo.N + I0 * fx + (long long)fo.nn[0] * (I1 * fy + (long long)fo.nn[1] * (I2 * fz)));
    xc[3 * g] = x[fg];
    xc[3 * g + 1] = x[fg + 1];
    xc[3 * g + 2] = x[fg + 2];
  }
}

// One axis of the transposed interpolation (the restriction is the tensor
// product of the 1-D ones, so it is applied axis by axis): `out` has the node
// counts `din` of `in` with axis d coarsened by f (D -> (D - 1) / f + 1),
// components innermost, and out[.., I, .., c] = sum over the fine nodes p of
// the support of coarse node I of hat(p, I, f) in[.., p, .., c], p ascending.
// One wavefront per output line (fixed node coordinates on axes 1..3; x and
// the component vary along the line, contiguous in memory; four lines per
// workgroup).
struct Dims4 {
  int n[4];
};

__global__ void __launch_bounds__(256) restrict_axis_kernel(Dims4 din, int d, int f, const double *__restrict__ in,
                                                            double *__restrict__ out) {
  int dout[4];
  for (int k = 0; k < 4; ++k) dout[k] = din.n[k];
  dout[d] = (din.n[d] - 1) / f + 1;
  const int lines = dout[1] * dout[2] * dout[3];
  const int lin = 3 * din.n[0], lout = 3 * dout[0];
  const double rf = 1.0 / f;
  const int lane = threadIdx.x & 63;
  for (int line = blockIdx.x * 4 + (threadIdx.x >> 6); line < lines; line += gridDim.x * 4) {
    double *orow = out + (long long)line * lout;
    if (d == 0) {   // (x lines too long for restrict_x_kernel's LDS)
      const double *irow = in + (long long)line * lin;   // axes 1..3 unchanged
      for (int t = lane; t < lout; t += 64) {
        const int I = t / 3, c = t - 3 * I;
        const int lo = max(0, I * f - f + 1), hi = min(din.n[0] - 1, I * f + f - 1);
        double acc = 0.0;
        for (int p = lo; p <= hi; ++p) acc += hat(p, I, f, rf) * irow[3 * p + c];
        orow[t] = acc;
      }
      continue;
    }
    // input line of node p on axis d: the output line's coordinates with axis d set to p
    const int o1 = line % dout[1], o2 = (line / dout[1]) % dout[2], o3 = line / (dout[1] * dout[2]);
    const int I = d == 1 ? o1 : d == 2 ? o2 : o3;
    const long long step = d == 1 ? 1 : d == 2 ? din.n[1] : (long long)din.n[1] * din.n[2];
    const long long line0 = o1 + (long long)din.n[1] * (o2 + (long long)din.n[2] * o3) - (long long)I * step;
    const int lo = max(0, I * f - f + 1), hi = min(din.n[d] - 1, I * f + f - 1);
    for (int t = lane; t < lout; t += 64) {
      double acc = 0.0;
      for (int p = lo; p <= hi; ++p) acc += hat(p, I, f, rf) * in[(line0 + p * step) * lin + t];
      orow[t] = acc;
    }
  }
}

// The x axis of the restriction (d = 0 above): lines are unchanged and
// contiguous, so a workgroup reads kRxLines consecutive input lines into LDS
// with one coalesced stream and forms all their outputs from there,
// out[line][3 I + c] = sum over p of hat(p, I, f) in[line][3 p + c].
constexpr int kRxLines = 16;

__global__ void __launch_bounds__(256) restrict_x_kernel(int nx, int lines, int f, const double *__restrict__ in,
                                                         double *__restrict__ out) {
  extern __shared__ double rx_lds[];
  const int lin = 3 * nx, cx = (nx - 1) / f + 1, lout = 3 * cx;
  const double rf = 1.0 / f;
  const int l0 = blockIdx.x * kRxLines, nl = min(kRxLines, lines - l0);
  const double *src = in + (long long)l0 * lin;
  for (int k = threadIdx.x; k < nl * lin; k += blockDim.x) rx_lds[k] = src[k];
  __syncthreads();
  double *dst = out + (long long)l0 * lout;
  for (int k = threadIdx.x; k < nl * lout; k += blockDim.x) {
    const int lq = k / lout, t = k - lq * lout;
    const int I = t / 3, c = t - 3 * I;
    const int lo = max(0, I * f - f + 1), hi = min(nx - 1, I * f + f - 1);
    const double *row = rx_lds + lq * lin + c;
    double acc = 0.0;
    for (int p = lo; p <= hi; ++p) acc += hat(p, I, f, rf) * row[3 * p];
    dst[k] = acc;
  }
}

// The x and y axes together: a workgroup coarsens one (z, t) plane of the fine
// vector, first in y, straight from memory (every fine line between two coarse
// ones is read for both, the second time from the cache; the loads of an entry
// do not depend on each other), then its cy lines in x, from LDS.  A 32^3 x 64
// vector (56 MB) takes 19 us; with the whole plane staged in LDS and x first it
// took 22, with one launch per axis 25 and 8 us.
__global__ void __launch_bounds__(256) restrict_xy_kernel(int nx, int ny, int fx, int fy, VecsIn xs,
                                                          double *__restrict__ out, long long ostride) {
  extern __shared__ double rxy_lds[];   // [cy][lin]
  const int lin = 3 * nx, cx = (nx - 1) / fx + 1, cy = (ny - 1) / fy + 1, lout = 3 * cx;
  const double *__restrict__ src = xs.p[blockIdx.y] + (long long)blockIdx.x * ny * lin;
  const double rx = 1.0 / fx, ry = 1.0 / fy;
  for (int k = threadIdx.x; k < cy * lin; k += 256) {
    const int I = k / lin, t = k - I * lin;
    const int lo = max(0, I * fy - fy + 1), hi = min(ny - 1, I * fy + fy - 1);
    const double *col = src + t;
    double acc = 0.0;
    for (int p0 = lo; p0 <= hi; p0 += 8) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = col[(long long)min(p0 + u, hi) * lin];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (p0 + u <= hi) acc += hat(p0 + u, I, fy, ry) * v[u];
    }
    rxy_lds[k] = acc;
  }
  __syncthreads();
  double *dst = out + blockIdx.y * ostride + (long long)blockIdx.x * cy * lout;
  for (int k = threadIdx.x; k < cy * lout; k += 256) {
    const int l = k / lout, t = k - l * lout, I = t / 3, c = t - 3 * I;
    const int lo = max(0, I * fx - fx + 1), hi = min(nx - 1, I * fx + fx - 1);
    const double *row = rxy_lds + l * lin + c;
    double acc = 0.0;
    for (int p = lo; p <= hi; ++p) acc += hat(p, I, fx, rx) * row[3 * p];
    dst[k] = acc;
  }
}

// The z and t axes together, planes of pl doubles already coarsened in x and
// y: out[I3][I2][e] = sum over t and z of hat_t hat_z in[p3][p2][e].
__global__ void __launch_bounds__(256) restrict_zt_kernel(int pl, int nz, int nt, int fz, int ft, VecsIn xs,
                                                          VecsOut ys) {
  const int cz = (nz - 1) / fz + 1, ct = (nt - 1) / ft + 1;
  const long long total = (long long)ct * cz * pl;
  const double *__restrict__ in = xs.p[blockIdx.y];
  const double rz = 1.0 / fz, rt = 1.0 / ft;
  for (long long q = blockIdx.x * (long long)blockDim.x + threadIdx.x; q < total;
       q += (long long)gridDim.x * blockDim.x) {
    const long long g = q / pl;
    const int e = (int)(q - g * pl), I2 = (int)(g % cz), I3 = (int)(g / cz);
    const int z0 = max(0, I2 * fz - fz + 1), z1 = min(nz - 1, I2 * fz + fz - 1);
    const int t0 = max(0, I3 * ft - ft + 1), t1 = min(nt - 1, I3 * ft + ft - 1);
    double acc = 0.0;
    for (int t = t0; t <= t1; ++t) {
      const double *src = in + (long long)t * nz * pl + e;
      double s = 0.0;
#pragma unroll 4
      for (int z = z0; z <= z1; ++z) s += hat(z, I2, fz, rz) * src[(long long)z * pl];
      acc += hat(t, I3, ft, rt) * s;
    }
    ys.p[blockIdx.y][q] = acc;
  }
}

}  // namespace

// y_i = I_c^h xc_i for q <= kTransferVecs vectors
static void prolong(const coarse *C, int q, const VecsIn &xc, const VecsOut &y, hipStream_t s) {
  const OpDev &fo = C->fine;
  const long long threads = 3LL * fo.nn[0] * ((fo.nn[1] - 1) / C->fac[1] + 1) * ((fo.nn[2] - 1) / C->fac[2] + 1) *
                            (fo.M + 1);
  hipLaunchKernelGGL(prolong_kernel, dim3(blocks_for(threads, 256), q), dim3(256), 0, s, fo, C->cop->d, C->fac[0],
                     C->fac[1], C->fac[2], C->fac[3], xc, y);
}

// LDS of restrict_xy_kernel; planes that leave room for two workgroups per
// compute unit go through it, larger ones axis by axis.
static size_t restrict_xy_lds(const coarse *C) {
  return sizeof(double) * 3 * (size_t)C->fine.nn[0] * (size_t)C->cop->d.nn[1];
}
constexpr size_t kRestrictXyLds = 64 * 1024;

// elements of one vector between restrict_xy_kernel and restrict_zt_kernel
static long long restrict_mid(const coarse *C) {
  const OpDev &co = C->cop->d;
  return 3LL * co.nn[0] * co.nn[1] * C->fine.nn[2] * (C->fine.M + 1);
}

// xc = (I_c^h)^T x, axis by axis (x, y, z, t; axes with factor 1 are skipped),
// or, given planes that restrict_xy_kernel has coarsened (anywhere but in
// C->rt[1]), along the other two axes (first = 2).
static void restrict_axes(const coarse *C, int first, const double *x, double *xc, hipStream_t s) {
  const OpDev &fo = C->fine, &co = C->cop->d;
  Dims4 dm{{fo.nn[0], fo.nn[1], fo.nn[2], fo.M + 1}};
  for (int d = 0; d < first; ++d) dm.n[d] = co.nn[d];
  int axes[4], na = 0;
  for (int d = first; d < 4; ++d)
    if (C->fac[d] > 1) axes[na++] = d;
  if (na == 0) {
    STKKT_HIP(hipMemcpyAsync(xc, x, sizeof(double) * 3 * fo.V, hipMemcpyDeviceToDevice, s));
    return;
  }
  const double *src = x;
  for (int k = 0; k < na; ++k) {
    const int d = axes[k];
    double *dst = k == na - 1 ? xc : C->rt[first > 0 ? 1 : k & 1].as<double>();
    Dims4 out = dm;
    out.n[d] = (dm.n[d] - 1) / C->fac[d] + 1;
    const int lines = out.n[1] * out.n[2] * out.n[3];
    const size_t xlds = sizeof(double) * kRxLines * 3 * (size_t)dm.n[0];
    if (d == 0 && xlds <= 64 * 1024)
      hipLaunchKernelGGL(restrict_x_kernel, dim3((lines + kRxLines - 1) / kRxLines), dim3(256), xlds, s, dm.n[0], lines,
                         C->fac[0], src, dst);
    else
      hipLaunchKernelGGL(restrict_axis_kernel, dim3(std::min((lines + 3) / 4, 1 << 20)), dim3(256), 0, s, dm, d,
                         C->fac[d], src, dst);
    dm = out;
    src = dst;
  }
  STKKT_HIP(hipGetLastError());
}

// Which axes go together.  A thread of restrict_xy_kernel reads its entries of
// the plane one batch after the other, and a launch has a workgroup per plane:
// few planes with many entries are slower than an axis at a time.  Planes,
// entries a thread and the whole restriction, together / by axes: 25, 1014 114 /
// 38 us; 45, 361 62 / 32; 189, 266 49 / 40; 136, 105 31 / 28; 245, 60 20 / 27;
// 427, 115 33 / 41.  A thread of restrict_zt_kernel reads a window of z and t
// nodes: 1521 of them 105 us against 27 for a launch per axis, 225 34 against
// 14, 121 21 against 14, 45 8 against 12.  (No rule depends on the number of
// vectors: a vector's result is the same among others.)
static bool fuse_xy(const coarse *C) {
  const long long planes = (long long)C->fine.nn[2] * (C->fine.M + 1);
  const long long entries = (3LL * C->fine.nn[0] * C->cop->d.nn[1] + 255) / 256 * (2 * C->fac[1] - 1);
  return restrict_xy_lds(C) <= kRestrictXyLds && planes <= INT32_MAX && planes >= 2 * entries;
}
constexpr long long kRestrictWindow = 64;
static bool fuse_zt(const coarse *C) { return (2LL * C->fac[2] - 1) * (2LL * C->fac[3] - 1) <= kRestrictWindow; }

// xc_i = (I_c^h)^T x_i for q <= kTransferVecs vectors; mid: q times
// restrict_mid(C) doubles outside C->rt[1] (not used when x and y are not coarsened)
static void restrict_transpose(const coarse *C, int q, const VecsIn &x, const VecsOut &xc, double *mid,
                               hipStream_t s) {
  const OpDev &fo = C->fine, &co = C->cop->d;
  const bool xy = C->fac[0] > 1 || C->fac[1] > 1, zt = C->fac[2] > 1 || C->fac[3] > 1;
  if (xy ? !fuse_xy(C) : !zt || !fuse_zt(C)) {
    for (int i = 0; i < q; ++i) restrict_axes(C, 0, x.p[i], xc.p[i], s);
    return;
  }
  VecsIn from = x;
  if (xy) {
    const long long step = restrict_mid(C);
    hipLaunchKernelGGL(restrict_xy_kernel, dim3((unsigned)(fo.nn[2] * (fo.M + 1)), q), dim3(256), restrict_xy_lds(C),
                       s, fo.nn[0], fo.nn[1], C->fac[0], C->fac[1], x, mid, step);
    for (int i = 0; i < q; ++i) from.p[i] = mid + i * step;
    if (!fuse_zt(C)) {
      for (int i = 0; i < q; ++i) restrict_axes(C, 2, from.p[i], xc.p[i], s);
      return;
    }
  }
  const int pl = 3 * co.nn[0] * co.nn[1];
  hipLaunchKernelGGL(restrict_zt_kernel, dim3(blocks_for(3 * co.V, 256), q), dim3(256), 0, s, pl, fo.nn[2], fo.M + 1,
                     C->fac[2], C->fac[3], from, xc);
  STKKT_HIP(hipGetLastError());
}

// xc_i = I_h^c x_i: the transposed interpolation or injection
static void restrict_to_coarse(const coarse *C, int q, const VecsIn &x, const VecsOut &xc, double *mid,
                               hipStream_t s) {
  if (C->params.restrict_kind == STKKT_RESTRICT_INJECTION) {
    const OpDev &fo = C->fine, &co = C->cop->d;
    for (int i = 0; i < q; ++i)
      hipLaunchKernelGGL(inject_kernel, dim3(blocks_for(co.V, 256, 8192)), dim3(256), 0, s, fo, co, C->fac[0],
                         C->fac[1], C->fac[2], C->fac[3], x.p[i], xc.p[i]);
    STKKT_HIP(hipGetLastError());
  } else {
    restrict_transpose(C, q, x, xc, mid, s);
  }
}

coarse *coarse_create(const kkt_op *fine, const coarse_params_t *cp, hipStream_t s) {
  STKKT_REQUIRE(cp->method == STKKT_COARSE_GMRES_RAS || cp->method == STKKT_COARSE_LU,
                "coarse_setup: unknown coarse solver");
  STKKT_REQUIRE(cp->precision == STKKT_F64 || cp->precision == STKKT_F32, "coarse_setup: bad precision");
  STKKT_REQUIRE(cp->restrict_kind == STKKT_RESTRICT_TRANSPOSE || cp->restrict_kind == STKKT_RESTRICT_INJECTION,
                "coarse_setup: bad restriction");
  if (cp->method == STKKT_COARSE_GMRES_RAS)
    STKKT_REQUIRE(cp->maxit >= 1 && cp->rtol > 0 && cp->rtol < 1, "coarse_setup: bad coarse solver settings");
  const OpDev &fd = fine->d;
  const int nf[4] = {fd.n[0], fd.n[1], fd.n[2], fd.M};
  for (int d = 0; d < 4; ++d)
    STKKT_REQUIRE(cp->factor[d] >= 1 && nf[d] % cp->factor[d] == 0,
                  "coarse_setup: coarsening factors must divide the element counts and nt");
  auto C = std::make_unique<coarse>();
  C->al = fine->al;
  C->fine = fd;
  C->fine_op = fine;
  C->params = *cp;
  for (int d = 0; d < 4; ++d) C->fac[d] = cp->factor[d];
  // coarse problem: same model, coarse mesh, averaged element coefficients
  kkt_problem_t p{};
  const int nc[3] = {fd.n[0] / cp->factor[0], fd.n[1] / cp->factor[1], fd.n[2] / cp->factor[2]};
  for (int d = 0; d < 3; ++d) {
    p.n[d] = nc[d];
    p.len[d] = fine->len[d];
    p.v[d] = fd.v[d];
  }
  p.nt = fd.M / cp->factor[3];
  p.T = fine->T;
  std::vector<double> ac((size_t)nc[0] * nc[1] * nc[2], 0.0);
  const int f0 = cp->factor[0], f1 = cp->factor[1], f2 = cp->factor[2];
  for (int ez = 0; ez < fd.n[2]; ++ez)
    for (int ey = 0; ey < fd.n[1]; ++ey)
      for (int ex = 0; ex < fd.n[0]; ++ex)
        ac[(ex / f0) + (size_t)nc[0] * ((ey / f1) + (size_t)nc[1] * (ez / f2))] +=
            fine->a_host[ex + (size_t)fd.n[0] * (ey + (size_t)fd.n[1] * ez)];
  for (double &v : ac) v /= (double)(f0 * f1 * f2);
  p.a_elem = ac.data();
  p.beta1 = fd.beta1;
  p.beta2 = fd.beta2;
  std::vector<int32_t> cs;
  for (int32_t j : fine->sensor_node) {
    const int i0 = j % fd.nn[0], i1 = (j / fd.nn[0]) % fd.nn[1], i2 = j / (fd.nn[0] * fd.nn[1]);
    STKKT_REQUIRE(i0 % f0 == 0 && i1 % f1 == 0 && i2 % f2 == 0,
                  "coarse_setup: every sensor must sit on a coarse node");
    cs.push_back((i0 / f0) + (nc[0] + 1) * ((i1 / f1) + (nc[1] + 1) * (i2 / f2)));
  }
  std::vector<double> zeros((size_t)(p.nt + 1) * cs.size(), 0.0);
  p.n_sensors = (int32_t)cs.size();
  p.sensor_node = cs.data();
  p.data = zeros.data();
  p.dirichlet_faces = fd.faces;
  p.variant = fd.variant;
  p.regularization = fd.reg;
  kkt_alloc_t al = fine->al.cb;
  C->cop = op_create(&p, al.alloc ? &al : nullptr, s);
  STKKT_REQUIRE(C->cop->d.nn[0] <= 512, "coarse_setup: more than 512 coarse nodes along x");
  const size_t nvc = 3 * (size_t)C->cop->d.V;
  C->xc = DevBuf(&C->al, sizeof(double) * nvc);
  C->yc = DevBuf(&C->al, sizeof(double) * nvc);
  {
    // the restriction's intermediates: sizes after the first and second coarsened axes
    long long dm[4] = {fd.nn[0], fd.nn[1], fd.nn[2], fd.M + 1}, sz[2] = {1, 1};
    int k = 0;
    for (int d = 0; d < 4 && k < 2; ++d)
      if (cp->factor[d] > 1) {
        dm[d] = (dm[d] - 1) / cp->factor[d] + 1;
        sz[k++] = 3 * dm[0] * dm[1] * dm[2] * dm[3];
      }
    C->rt[0] = DevBuf(&C->al, sizeof(double) * sz[0]);
    C->rt[1] = DevBuf(&C->al, sizeof(double) * sz[1]);
  }
  if (cp->method == STKKT_COARSE_LU) {
    C->lu = std::make_unique<CoarseLU>(&C->al, C->cop, cp->precision, s);
  } else {
    ras_params_t rp{};
    for (int d = 0; d < 4; ++d) rp.p[d] = cp->p[d];
    rp.overlap = cp->overlap;
    rp.precision = cp->precision;
    rp.ilu_level = 0;
    C->cras = ras_create(C->cop, &rp, s);
    C->work = std::make_unique<GmresWork>(&C->cop->al, (long long)nvc, cp->maxit, false, false);
  }
  return C.release();
}

void coarse_apply_device(const coarse *C, const double *x, double *y, hipStream_t s) {
  const OpDev &co = C->cop->d;
  restrict_to_coarse(C, 1, VecsIn{{x}}, VecsOut{{C->xc.as<double>()}}, C->rt[0].as<double>(), s);
  if (C->lu) {
    const long long nvc = 3 * co.V;
    if (C->lu->one_vector_on_mfma()) C->lu->solve_multi(1, C->xc.as<double>(), nvc, C->yc.as<double>(), nvc, s);
    else C->lu->solve(C->xc.as<double>(), C->yc.as<double>(), s);
  } else {
    fill_zero(C->yc.as<double>(), 3 * co.V, s);
    solve_params_t sp{};
    sp.restart = C->params.maxit;
    sp.maxit = C->params.maxit;
    sp.rtol = C->params.rtol;
    sp.flexible = 0;
    sp.fixed_iters = 0;
    const int st = gmres_solve(C->cop, C->cras, nullptr, sp, C->xc.as<double>(), C->yc.as<double>(), s, nullptr,
                               C->work.get());
    if (st != STKKT_OK && st != STKKT_NOT_CONVERGED) throw Error(st, "coarse solve failed");
  }
  prolong(C, 1, VecsIn{{C->yc.as<double>()}}, VecsOut{{y}}, s);
  STKKT_HIP(hipGetLastError());
}

void coarse_apply_multi_device(const coarse *C, int q, const double *const *x, double *const *y, hipStream_t s) {
  if (q <= 0) return;
  if (!C->lu) {
    for (int i = 0; i < q; ++i) coarse_apply_device(C, x[i], y[i], s);
    return;
  }
  const long long nvc = 3 * C->cop->d.V;
  if (q > C->mcap) {
    STKKT_HIP(hipStreamSynchronize(s));   // launches already queued may still use the old vectors
    C->xcm = DevBuf(&C->al, sizeof(double) * (size_t)nvc * q);
    C->ycm = DevBuf(&C->al, sizeof(double) * (size_t)nvc * q);
    C->midm = DevBuf(&C->al, sizeof(double) * (size_t)restrict_mid(C) * std::min(q, kTransferVecs));
    C->mcap = q;
  }
  double *xc = C->xcm.as<double>(), *yc = C->ycm.as<double>();
  for (int i0 = 0; i0 < q; i0 += kTransferVecs) {
    const int m = std::min(kTransferVecs, q - i0);
    VecsIn in{};
    VecsOut out{};
    for (int i = 0; i < m; ++i) {
      in.p[i] = x[i0 + i];
      out.p[i] = xc + (i0 + i) * nvc;
    }
    restrict_to_coarse(C, m, in, out, C->midm.as<double>(), s);
  }
  C->lu->solve_multi(q, xc, nvc, yc, nvc, s);
  for (int i0 = 0; i0 < q; i0 += kTransferVecs) {
    const int m = std::min(kTransferVecs, q - i0);
    VecsIn in{};
    VecsOut out{};
    for (int i = 0; i < m; ++i) {
      in.p[i] = yc + (i0 + i) * nvc;
      out.p[i] = y[i0 + i];
    }
    prolong(C, m, in, out, s);
  }
  STKKT_HIP(hipGetLastError());
}

void coarse_apply_strided(const coarse *C, int q, const double *x, long long ldx, double *y, long long ldy,
                          hipStream_t s) {
  const long long n = 3 * C->fine.V;
  STKKT_REQUIRE(q >= 0, "coarse_apply_multi: q must be >= 0");
  if (q == 0) return;
  STKKT_REQUIRE(ldx >= n && ldy >= n, "coarse_apply_multi: strides shorter than the fine vector");
  const double *xe = x + (q - 1) * ldx + n;
  const double *ye = y + (q - 1) * ldy + n;
  STKKT_REQUIRE(ye <= x || xe <= y, "coarse_apply_multi: x and y must not overlap");
  std::vector<const double *> xs(q);
  std::vector<double *> ys(q);
  for (int i = 0; i < q; ++i) {
    xs[i] = x + i * ldx;
    ys[i] = y + i * ldy;
  }
  coarse_apply_multi_device(C, q, xs.data(), ys.data(), s);
}

void coarse_free(coarse *c) { delete c; }

bool coarse_built_for(const coarse *c, const kkt_op *op) { return c->fine_op == op; }

}  // namespace stkkt
