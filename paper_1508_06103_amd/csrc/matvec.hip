// The operator application of the public entry point, in element modes.
#include <cmath>
#include <type_traits>
#include <vector>

#include "common.hpp"
#include "matvec_rows.hpp"
#include "stencil.hpp"

namespace stkkt {

// --------------------------------------------------------------------------
// y = F_h x, matrix-free.  Rows follow the block formula of kkt_block_c()
// regrouped by spatial operator.  With P_i = 0 on Dirichlet nodes and 1
// elsewhere, and per node i the combined fields
//   U1 = P (c^n - c^{n-1}) - tau/2 (f^{n-1} + f^n)       S1 = P (c^n + c^{n-1})
//   U2 = P (m g^n - p g^{n+1})                          S2 = P (m g^n + p g^{n+1})
//   U3 = beta1 (St f)^n - { DTO: tau/2 S2 ; OTD: P (Tt g)^n }   T3 = beta2 (Tt f)^n
//   (H1-L2 regularisation: beta2 (Tt f)^n is added to U3 instead and T3 = 0)
// (m = [n >= 1] for DTO and 1 for OTD, p = [n < M]; (St f)^n, (Tt f)^n the
// time stiffness / mass rows of level n), the rows of an interior node j are
//   C (n >= 1):  sum_i B_ji U1_i + tau/2 (A + N)_ji S1_i
//   G:           sum_i B_ji U2_i + tau/2 (A + N^T)_ji S2_i
//                + DTO: [n = 0] g_j^0 + w_n S_j c_j^n ; OTD (n < M): tau/2 S_j (c_j^n + c_j^{n+1})
//   f:           sum_i B_ji U3_i + K_ji T3_i
// and Dirichlet C/G rows, the C row of level 0 and the OTD G row of level M
// are identity rows.
//
// B, A, N and K are sums over elements, and on one element each is a tensor
// product of 2 x 2 matrices of its axes.  In the sum / difference modes of an
// axis, s = u_0 + u_1 and d = u_0 - u_1, with results r_0 = S + D, r_1 = S - D,
//   mass:        S = h/4 s,  D = h/12 d          stiffness:  D = d / h
//   convection:  S = -d / 2                      its transpose:  D = -s / 2
// so in the eight modes of an element mass and stiffness are diagonal (the
// element coefficient multiplies seven numbers) and convection couples modes in
// pairs.  End-of-mesh rules follow from the elements that exist.
//
// A workgroup owns a tile of (x, y) nodes at one time level and marches along
// z.  A thread is one node column with its halo, and the element column to its
// upper right.  Per plane it forms its node's six fields and puts them in LDS,
// reads those of its element's other three columns, takes the modes in x and
// y, pairs them with the previous plane's in z, multiplies, and turns the
// element's results back into corner values: the lower plane's are complete
// with the carry of the element below, and three of the four corners go
// through LDS to the columns that own them.  Both exchanges of consecutive
// planes share one barrier.  About 300 FP64 operations and 42 LDS doubles per
// column and plane; summing 27 neighbours per node from LDS took 162 LDS
// doubles and a table of 27 entries per node, and left the vector units idle
// two thirds of the time (cube48x96 581 us, this 307).
//
// In modes an infinite entry meets itself with both signs, and sums of eight
// values overflow before their weights bring them down.  Entries that come out
// non-finite are therefore formed again at the end of the march, as the sum
// over the neighbours: it alone decides what is infinite and what is not a
// number.
//
// The solvers keep matvec_device's form, the sum over 27 neighbours: a change
// in the order of the sums comes out of a long restarted solve with FP32
// preconditioners enlarged to 5e-9 of the solution (24^3 x 32, 145 steps).
// --------------------------------------------------------------------------
namespace {

constexpr int kMvThreads = 256;
// LDS per thread: two buffers of three field pairs and of nine corner values
constexpr size_t kMvLds = 2 * (3 * sizeof(double2) + 9 * sizeof(double)) * kMvThreads;

// Mesh and time constants of the matvec, formed on the host.  Mode index of a
// plane: bit 0 the x mode, bit 1 the y mode (0 = s, 1 = d); [z mode][plane mode].
struct MvModes {
  double M[2][4], K[2][4];            // mass and stiffness of a mode
  double Nx[2][2], Ny[2][2], Nz[4];   // tau/2 x convection: [z][y], [z][x], [plane] of the modes that stay
  // rows of the time stiffness St and mass Tt on the first, an inner and the
  // last level: (n, n - 1), (n, n), (n, n + 1); trapezoid weight
  struct Level {
    double st[3], tt[3], wn, pad;
  } lv[3];
  double ht, beta1, beta2;
  int l2, pad;   // H1-L2 regularisation: beta2 (Tt f) joins U3 (mass) instead of T3 (stiffness)
  // of the sum over neighbours
  MvConst sums;
  OpDev op;
  const double *atab;
};

MvModes make_mv_modes(const OpDev &d, const double *atab) {
  MvModes c{};
  double m[3][2], k[3][2];
  for (int a = 0; a < 3; ++a) {
    m[a][0] = d.h[a] / 4.0;
    m[a][1] = d.h[a] / 12.0;
    k[a][0] = 0.0;
    k[a][1] = 1.0 / d.h[a];
  }
  c.ht = 0.5 * d.tau;
  for (int z = 0; z < 2; ++z)
    for (int q = 0; q < 4; ++q) {
      const int x = q & 1, y = q >> 1;
      c.M[z][q] = m[0][x] * m[1][y] * m[2][z];
      c.K[z][q] = k[0][x] * m[1][y] * m[2][z] + m[0][x] * k[1][y] * m[2][z] + m[0][x] * m[1][y] * k[2][z];
    }
  for (int z = 0; z < 2; ++z)
    for (int i = 0; i < 2; ++i) {
      c.Nx[z][i] = -0.5 * c.ht * d.v[0] * m[1][i] * m[2][z];
      c.Ny[z][i] = -0.5 * c.ht * d.v[1] * m[0][i] * m[2][z];
    }
  for (int q = 0; q < 4; ++q) c.Nz[q] = -0.5 * c.ht * d.v[2] * m[0][q & 1] * m[1][q >> 1];
  for (int e = 0; e < 3; ++e) {
    const double it = 1.0 / d.tau;
    MvModes::Level &l = c.lv[e];
    l.st[0] = e == 0 ? 0.0 : -it;
    l.st[1] = e == 1 ? 2.0 * it : it;
    l.st[2] = e == 2 ? 0.0 : -it;
    l.tt[0] = e == 0 ? 0.0 : d.tau / 6.0;
    l.tt[1] = e == 1 ? 2.0 * (d.tau / 3.0) : d.tau / 3.0;
    l.tt[2] = e == 2 ? 0.0 : d.tau / 6.0;
    l.wn = e == 1 ? d.tau : c.ht;
  }
  c.beta1 = d.beta1;
  c.beta2 = d.beta2;
  c.l2 = d.reg == STKKT_REG_H1L2;
  c.sums = make_mv_const(d);
  c.op = d;
  c.atab = atab;
  return c;
}

typedef double mv_d2 __attribute__((ext_vector_type(2), aligned(8)));

// Modes of one field on an element's face from its nodal values at (0,0),
// (1,0), (0,1), (1,1).
__device__ inline void face_modes(double a, double b, double c, double e, double (&m)[4]) {
  const double s0 = a + b, d0 = a - b, s1 = c + e, d1 = c - e;
  m[0] = s0 + s1;
  m[1] = d0 + d1;
  m[2] = s0 - s1;
  m[3] = d0 - d1;
}

// Row (n, j), j = (jx, jy, jz), of y as the sum over the neighbours; xn and yn:
// level n of x and y.
__device__ inline void row_by_neighbours(const OpDev &op, const MvConst &mc, const double *__restrict__ atab,
                                         const double *__restrict__ xn, double *yn, int n, int jx, int jy,
                                         int jz) {
  const int M = op.M;
  const long long N = op.N, j = jx + (long long)op.nn[0] * (jy + (long long)op.nn[1] * jz);
  const bool dto = op.variant == STKKT_DTO, hm = n >= 1, hp = n < M, tend = !hm || !hp;
  const double stm = hm ? -mc.inv_tau : 0.0, st0 = tend ? mc.inv_tau : 2.0 * mc.inv_tau, stp = hp ? -mc.inv_tau : 0.0;
  const double ttm = hm ? mc.tau6 : 0.0, tt0 = tend ? mc.tau3 : 2.0 * mc.tau3, ttp = hp ? mc.tau6 : 0.0;
  auto at = [&](int dy, int dz, double2 (&r)[9]) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const int gx = jx + i - 1, gy = jy + dy, gz = jz + dz;
      r[3 * i] = r[3 * i + 1] = r[3 * i + 2] = make_double2(0.0, 0.0);
      if (gx < 0 || gx >= op.nn[0] || gy < 0 || gy >= op.nn[1] || gz < 0 || gz >= op.nn[2]) continue;
      const double *p0 = xn + 3 * (gx + (long long)op.nn[0] * (gy + (long long)op.nn[1] * gz));
      const double *pm = hm ? p0 - 3 * N : p0, *pp = hp ? p0 + 3 * N : p0;
      const double P = on_dirichlet(op, gx, gy, gz) ? 0.0 : 1.0;
      const double cm = hm ? pm[0] : 0.0, gm = hm ? pm[1] : 0.0, fm = hm ? pm[2] : 0.0;
      const double gp = hp ? pp[1] : 0.0, fp = hp ? pp[2] : 0.0;
      const double c0 = p0[0], g0 = p0[1], f0 = p0[2], gn = !dto || hm ? g0 : 0.0;
      const double S2 = P * (gn + gp), ttf = mc.beta2 * (ttm * fm + tt0 * f0 + ttp * fp);
      const double U3 = mc.beta1 * (stm * fm + st0 * f0 + stp * fp) -
                        (dto ? mc.ht * S2 : P * (ttm * gm + tt0 * g0 + ttp * gp));
      r[3 * i] = make_double2(P * (c0 - cm) - mc.ht * (fm + f0), P * (c0 + cm));
      r[3 * i + 1] = make_double2(P * (gn - gp), S2);
      r[3 * i + 2] = mc.l2 ? make_double2(U3 + ttf, 0.0) : make_double2(U3, ttf);
    }
  };
  const RowSums q = neighbour_sums(mc, axis_centre(mc, 0, jx, op.nn[0]), axis_centre(mc, 1, jy, op.nn[1]),
                                   axis_centre(mc, 2, jz, op.nn[2]), atab + 27 * j, at);
  const bool Pj = !on_dirichlet(op, jx, jy, jz);
  const double sens = op.sensor[j], cj = xn[3 * j], gj = xn[3 * j + 1];
  double *ys = yn + 3 * j;
  ys[0] = (n == 0 || !Pj) ? cj : q.aC + mc.ht * q.sC;
  double g = gj;
  if (Pj && dto) g = q.aG + mc.ht * q.sG + (n == 0 ? gj : 0.0) + (tend ? mc.ht : 2.0 * mc.ht) * sens * cj;
  else if (Pj && hp) g = q.aG + mc.ht * q.sG + mc.ht * sens * (cj + xn[3 * (N + j)]);
  ys[1] = g;
  ys[2] = q.aF;
}

// One (tile, z chunk, time level) work item w of one operator.  The constants
// are read again every plane (scalar loads): kept in scalar registers they
// spill to vector lanes.
template <int T>
__device__ inline void march_item(const OpDev &op, const MvMarch &tl, const MvModes *modes,
                                  const double *__restrict__ x, double *y, int w) {
  extern __shared__ double2 mv_lds[];
  // what the end of the march needs again waits in memory: scalar registers are short during it
  __shared__ struct {
    const double *x;
    double *y;
    int n, z0, z1;
  } late;
  const cptr<MvModes> mc = as_const(modes);
  const int t = (int)threadIdx.x;
  const int M = op.M, nlev = M + 1;
  const int n = w % nlev, item = w / nlev, tile = item % tl.ntiles, zc = item / tl.ntiles;
  const int nn0 = op.nn[0], nn1 = op.nn[1], nn2 = op.nn[2];
  const int z0 = zc * tl.zlen, z1 = min(nn2, z0 + tl.zlen);   // planes written
  const int pa = max(z0 - 1, 0), pb = min(z1, nn2 - 1);       // planes whose fields are needed
  const int hx = tl.t[0] + 2, hy = tl.t[1] + 2;
  const int tx = t % hx, ty = t / hx;
  const int gx = (tile % tl.nt[0]) * tl.t[0] - 1 + tx, gy = (tile / tl.nt[0]) * tl.t[1] - 1 + ty;
  const int cx = min(max(gx, 0), nn0 - 1), cy = min(max(gy, 0), nn1 - 1);
  const bool elem = tx + 1 < hx && ty + 1 < hy && gx >= 0 && gx < op.n[0] && gy >= 0 && gy < op.n[1];
  const bool own = tx >= 1 && tx + 1 < hx && ty >= 1 && ty + 1 < hy && gx < nn0 && gy < nn1;
  const bool dto = op.variant == STKKT_DTO;
  const bool hm = n >= 1, hp = n < M;
  const bool mflag = !dto || hm;
  const cptr<MvModes::Level> lv = &mc->lv[hm ? (hp ? 1 : 2) : 0];
  const double st0 = lv->st[0], st1 = lv->st[1], st2 = lv->st[2], tt0 = lv->tt[0], tt1 = lv->tt[1], tt2 = lv->tt[2];
  const double ht = mc->ht, beta1 = mc->beta1, beta2 = mc->beta2, wn = lv->wn;
  const bool l2 = mc->l2 != 0;
  const long long plane = 3LL * nn0 * nn1, level = 3LL * op.N;
  // uniform bases of the plane at levels n - 1, n, n + 1; the thread's byte
  // offsets in a plane of x, of sensor, and in an element layer (clamped into the mesh)
  const long long vs = 8 * ((long long)cy * nn0 + cx), vo = 3 * vs;
  const long long vae = 8 * ((long long)min(cy, op.n[1] - 1) * op.n[0] + min(cx, op.n[0] - 1));
  const double *b0 = x + n * level, *bm = hm ? b0 - level : b0, *bp = hp ? b0 + level : b0;
  const long long aplane = (long long)op.n[0] * op.n[1];
  const bool side = ((op.faces & 1u) && gx == 0) || ((op.faces & 2u) && gx == nn0 - 1) || ((op.faces & 4u) && gy == 0) ||
                    ((op.faces & 8u) && gy == nn1 - 1);
  auto dirichlet = [&](int p) {
    return side || ((op.faces & 16u) && p == 0) || ((op.faces & 32u) && p == nn2 - 1);
  };
  // LDS: two buffers of [3][T] field pairs, two of [9][T] corner values.  The
  // neighbours' places are clamped where there is no neighbour (unused then).
  if (t == 0) {   // (read after the barriers of the planes)
    late.x = x;
    late.y = y;
    late.n = n;
    late.z0 = z0;
    late.z1 = z1;
  }
  double2 *const fb0 = mv_lds;
  double *const cb0 = reinterpret_cast<double *>(mv_lds + 6 * T);
  const int tr = min(t + 1, T - 1), tu = min(t + hx, T - 1), tur = min(t + hx + 1, T - 1);
  const int tl1 = max(t - 1, 0), td = max(t - hx, 0), tdl = max(t - hx - 1, 0);

  mv_d2 rm, r0, rp;        // (c, g) of the requested plane at levels n - 1, n, n + 1
  double fm, f0, fp, a_e;  // f, and the coefficient of the element layer below it
  double sens;             // sensor mask of the plane written when the requested one is taken
  auto request = [&](int p) {
    const int ps = min(max(p - 2, 0), nn2 - 1);   // (the last request of a march is past the planes it writes)
    sens = *reinterpret_cast<const double *>(reinterpret_cast<const char *>(op.sensor + ps * (plane / 3)) + vs);
    const int q = min(p, pb);
    const char *pm = reinterpret_cast<const char *>(bm + q * plane), *p0 = reinterpret_cast<const char *>(b0 + q * plane),
               *pp = reinterpret_cast<const char *>(bp + q * plane);
    rm = *reinterpret_cast<const mv_d2 *>(pm + vo);
    fm = *reinterpret_cast<const double *>(pm + vo + 16);
    r0 = *reinterpret_cast<const mv_d2 *>(p0 + vo);
    f0 = *reinterpret_cast<const double *>(p0 + vo + 16);
    rp = *reinterpret_cast<const mv_d2 *>(pp + vo);
    fp = *reinterpret_cast<const double *>(pp + vo + 16);
    a_e = *reinterpret_cast<const double *>(reinterpret_cast<const char *>(op.a_elem + max(q - 1, 0) * aplane) + vae);
  };
  double X[6][4];   // face modes of the last plane: U1, S1, U2, S2, U3, T3
  double carry[3][4], corner[3][3], mine[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    mine[k] = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) X[2 * k][q] = X[2 * k + 1][q] = carry[k][q] = 0.0;
#pragma unroll
    for (int q = 0; q < 3; ++q) corner[k][q] = 0.0;
  }
  // node values needed when the plane is written, two planes later: c, g, and
  // c^{n+1} (OTD sensor term)
  double c_a = 0.0, g_a = 0.0, e_a = 0.0, c_b = 0.0, g_b = 0.0, e_b = 0.0;
  double check = 0.0;   // not a number once a value written is not finite
  // Plane p.  kFields: its fields are needed (p <= pb); kLayer: the element
  // layer between planes p - 1 and p exists (pa < p <= pb); par: (p - pa) & 1.
  auto plane_step = [&](int p, auto kf, auto kl, auto par) {
    constexpr bool kFields = decltype(kf)::value, kLayer = decltype(kl)::value;
    cptr<MvModes> m = mc;
    asm volatile("" : "+s"(m));
    double2 *const fb = fb0 + par * (3 * T);
    double *const cb = cb0 + par * (9 * T);
    const double a_l = ht * a_e, sens_o = sens;
    const double cn = r0.x, gr = r0.y, en = rp.x;
    if (kFields) {
      const bool dn = dirichlet(p);
      const double cm = hm ? rm.x : 0.0, gm = hm ? rm.y : 0.0, fmv = hm ? fm : 0.0;
      const double gn = mflag ? gr : 0.0, gp = hp ? rp.y : 0.0, fpv = hp ? fp : 0.0;
      const double P = dn ? 0.0 : 1.0, S2 = P * (gn + gp);
      const double stf = st0 * fmv + st1 * f0 + st2 * fpv;
      const double ttf = beta2 * (tt0 * fmv + tt1 * f0 + tt2 * fpv);
      double U3 = beta1 * stf;
      if (dto) U3 -= ht * S2;
      else U3 -= P * (tt0 * gm + tt1 * gr + tt2 * gp);
      fb[t] = make_double2(P * (cn - cm) - ht * (fmv + f0), P * (cn + cm));
      fb[T + t] = make_double2(P * (gn - gp), S2);
      fb[2 * T + t] = l2 ? make_double2(U3 + ttf, 0.0) : make_double2(U3, ttf);
    }
    // corners of plane p - 2 that belong to other columns
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int q = 0; q < 3; ++q) cb[(3 * k + q) * T + t] = corner[k][q];
    const double keep0 = mine[0], keep1 = mine[1], keep2 = mine[2];   // its own corner of plane p - 2
    const double c_o = c_b, g_o = g_b, e_o = e_b;
    c_b = c_a, g_b = g_a, e_b = e_a;
    c_a = cn, g_a = gr, e_a = en;
    request(p + 1);
    __syncthreads();
    if (elem) {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        double tot[4];
        if (kFields) {
          const double2 v0 = fb[k * T + t], v1 = fb[k * T + tr], v2 = fb[k * T + tu], v3 = fb[k * T + tur];
          double u[4], v[4];
          face_modes(v0.x, v1.x, v2.x, v3.x, u);
          face_modes(v0.y, v1.y, v2.y, v3.y, v);
          if (kLayer) {
            double O[2][4], S[2][4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              O[0][q] = m->M[0][q] * (X[2 * k][q] + u[q]);
              O[1][q] = m->M[1][q] * (X[2 * k][q] - u[q]);
              S[0][q] = X[2 * k + 1][q] + v[q];
              S[1][q] = X[2 * k + 1][q] - v[q];
            }
#pragma unroll
            for (int z = 0; z < 2; ++z)
#pragma unroll
              for (int q = 0; q < 4; ++q)
                if (z + q > 0) {
                  const double ks = m->K[z][q] * S[z][q];
                  O[z][q] += k == 2 ? ks : a_l * ks;
                }
            // convection: k = 0 takes difference modes to sum modes, k = 1 (its transpose) the other way
            if (k < 2) {
#pragma unroll
              for (int z = 0; z < 2; ++z)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                  const int sx = 2 * i, dx = 2 * i + 1, sy = i, dy = i + 2;
                  O[z][k == 0 ? sx : dx] += m->Nx[z][i] * S[z][k == 0 ? dx : sx];
                  O[z][k == 0 ? sy : dy] += m->Ny[z][i] * S[z][k == 0 ? dy : sy];
                }
#pragma unroll
              for (int q = 0; q < 4; ++q) O[k][q] += m->Nz[q] * S[1 - k][q];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              tot[q] = carry[k][q] + (O[0][q] + O[1][q]);
              carry[k][q] = O[0][q] - O[1][q];
            }
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            X[2 * k][q] = u[q];
            X[2 * k + 1][q] = v[q];
          }
        }
        if (!kLayer) {   // first plane: nothing below it; past the last plane: nothing above it
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            tot[q] = carry[k][q];
            carry[k][q] = 0.0;
          }
        }
        // corner values of plane p - 1
        const double ss = tot[0] + tot[2], sd = tot[0] - tot[2], ds = tot[1] + tot[3], dd = tot[1] - tot[3];
        mine[k] = ss + ds;
        corner[k][0] = ss - ds;   // (1, 0)
        corner[k][1] = sd + dd;   // (0, 1)
        corner[k][2] = sd - dd;   // (1, 1)
      }
    }
    const int o = p - 2;
    if (own && o >= z0 && o < z1) {
      const double q0 = keep0 + cb[tl1] + (cb[T + td] + cb[2 * T + tdl]);
      const double q1 = keep1 + cb[3 * T + tl1] + (cb[4 * T + td] + cb[5 * T + tdl]);
      const double q2 = keep2 + cb[6 * T + tl1] + (cb[7 * T + td] + cb[8 * T + tdl]);
      const bool dn = dirichlet(o);
      double g;
      if (dn) {
        g = g_o;
      } else if (dto) {
        g = q1 + (hm ? 0.0 : g_o) + wn * sens_o * c_o;
      } else {
        g = hp ? q1 + ht * sens_o * (c_o + e_o) : g_o;
      }
      char *ys = reinterpret_cast<char *>(y + n * level + o * plane);
      const double c = (!hm || dn) ? c_o : q0;
      check = __builtin_fma(c, 0.0, __builtin_fma(g, 0.0, __builtin_fma(q2, 0.0, check)));
      *reinterpret_cast<mv_d2 *>(ys + vo) = mv_d2{c, g};
      *reinterpret_cast<double *>(ys + vo + 16) = q2;
    }
  };
  request(pa);
  using Even = std::integral_constant<int, 0>;
  using Odd = std::integral_constant<int, 1>;
  plane_step(pa, std::true_type{}, std::false_type{}, Even{});
  int p = pa + 1;
  for (; p + 1 <= pb; p += 2) {
    plane_step(p, std::true_type{}, std::true_type{}, Odd{});
    plane_step(p + 1, std::true_type{}, std::true_type{}, Even{});
  }
  if (p <= pb) {
    plane_step(p, std::true_type{}, std::true_type{}, Odd{});
    ++p;
  }
#pragma unroll 1
  for (; p <= z1 + 1; ++p) plane_step(p, std::false_type{}, std::false_type{}, (p - pa) & 1);
  if (check != check) {
    const MvConst sums = load_uniform(&modes->sums);
    const OpDev full = load_uniform(&modes->op);
    const int nl = late.n, ze = late.z1;
    const double *xn = late.x + nl * 3LL * full.N;
    double *yn = late.y + nl * 3LL * full.N;
#pragma unroll 1
    for (int z = late.z0; z < ze; ++z) {
      const double *ys = yn + 3 * (gx + (long long)full.nn[0] * (gy + (long long)full.nn[1] * z));
      if (!std::isfinite(ys[0]) || !std::isfinite(ys[1]) || !std::isfinite(ys[2]))
        row_by_neighbours(full, sums, modes->atab, xn, yn, nl, gx, gy, z);
    }
  }
}

template <int T>
__global__ void __launch_bounds__(T, 2) matvec_march_kernel(OpDev op, MvMarch tl, const MvModes *__restrict__ mc,
                                                            const double *__restrict__ x, double *y) {
  march_item<T>(op, tl, mc, x, y, xcd_work_index());
}

}  // namespace

// Tile of owned (x, y) nodes, at most kMvThreads columns with the halo: the
// fewest wavefronts over the mesh, wide lines first.  z is cut so that about
// 1024 workgroups exist (two per compute unit, twice), at a cost of three
// planes of overhead per cut.
MvMarch choose_matvec_march(const OpDev &d) {
  MvMarch best{};
  long long best_cost = -1;
  for (int tx = 1; tx <= std::min(d.nn[0], kMvThreads / 3 - 2); ++tx)
    for (int ty = 1; ty <= std::min(d.nn[1], kMvThreads / (tx + 2) - 2); ++ty) {
      const int cols = (tx + 2) * (ty + 2);
      const int ntx = (d.nn[0] + tx - 1) / tx, nty = (d.nn[1] + ty - 1) / ty;
      // columns, counted in wavefronts
      const long long cost = (long long)ntx * nty * ((cols + 63) / 64);
      if (best_cost < 0 || cost <= best_cost) {
        best_cost = cost;
        best.t[0] = tx;
        best.t[1] = ty;
        best.nt[0] = ntx;
        best.nt[1] = nty;
        best.threads = (cols + 63) / 64 * 64;
      }
    }
  best.ntiles = best.nt[0] * best.nt[1];
  const long long per = (long long)best.ntiles * (d.M + 1);
  const int cuts = (int)std::max<long long>(1, std::min<long long>(d.nn[2], (1024 + per - 1) / per));
  best.zlen = (d.nn[2] + cuts - 1) / cuts;
  best.nz = (d.nn[2] + best.zlen - 1) / best.zlen;
  // Thin meshes: a plane costs a wavefront about 1.8 us however few of its lanes
  // own a node, so long marches of few columns are slower than the sum over
  // neighbours.  Columns, planes a march: march / sum in us.  4, 3 12.4 / 9.5 (31
  // planes, 97 levels); 9, 5 16.4 / 11.0; 12, 3 12.4 / 10.6; 16, 6 17 / 15; 16, 28
  // 58 / 41; 20, 28 58 / 49; 25, 28 58 / 53.  The other side: 9, 2 8.3 / 9.3; 16,
  // 5 12 / 15; 25, 17 38 / 46; 35, 28 58 / 69.
  const int columns = d.nn[0] * d.nn[1];
  best.sums = best.zlen > (columns <= 12 ? 2 : columns <= 16 ? 5 : columns <= 26 ? 24 : d.nn[2]);
  return best;
}

void matvec_constants(kkt_op *op, hipStream_t s) {
  const MvModes c = make_mv_modes(op->d, op->atab.as<double>());
  const char *p = reinterpret_cast<const char *>(&c);
  op->mvc_host.assign(p, p + sizeof(c));
  op->mvc = DevBuf(&op->al, sizeof(c));
  STKKT_HIP(hipMemcpyAsync(op->mvc.ptr, op->mvc_host.data(), sizeof(c), hipMemcpyHostToDevice, s));
}

static long long matvec_items(const OpDev &d, const MvMarch &tl) { return (long long)tl.ntiles * tl.nz * (d.M + 1); }
static size_t matvec_lds(int threads) { return kMvLds / kMvThreads * (size_t)threads; }

void matvec_march_device(const kkt_op *op, const double *x, double *y, hipStream_t s) {
  if (op->mvm.sums) {
    matvec_device(op, x, y, s);
    return;
  }
  const OpDev &d = op->d;
  const long long grid = matvec_items(d, op->mvm);
  if (grid > INT32_MAX) throw Error(STKKT_EINVAL, "kkt_matvec: mesh too large");
  const auto kernel = op->mvm.threads == 64    ? matvec_march_kernel<64>
                      : op->mvm.threads == 128 ? matvec_march_kernel<128>
                      : op->mvm.threads == 192 ? matvec_march_kernel<192>
                                              : matvec_march_kernel<256>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(op->mvm.threads), matvec_lds(op->mvm.threads), s, d, op->mvm,
                     op->mvc.as<MvModes>(), x, y);
  STKKT_HIP(hipGetLastError());
}

}  // namespace stkkt
