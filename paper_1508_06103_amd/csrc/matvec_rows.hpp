// The rows of F_h as sums over the 27 spatial neighbours: the constants and the
// sum itself, shared by the solvers' operator and by the public one.
#pragma once

#include "common.hpp"

namespace stkkt {

// Mesh and time constants of the matvec, formed on the host so that the
// kernel never evaluates a product of uniform values in vector registers.
struct MvConst {
  double h6[3], hinv[3];   // h/6 and 1/h per axis (off-centre mass, -stiffness)
  double v[3];
  double cyz[2][2][4];     // corner rows (dy, dz = +-1): myz, kyz, nyz, v0 myz
  double ht, inv_tau, tau6, tau3, beta1, beta2;
  int l2;   // H1-L2 regularisation: beta2 (Tt f) joins U3 (mass) instead of T3 (stiffness)
};

inline MvConst make_mv_const(const OpDev &d) {
  MvConst c{};
  for (int a = 0; a < 3; ++a) {
    c.h6[a] = d.h[a] / 6.0;
    c.hinv[a] = 1.0 / d.h[a];
    c.v[a] = d.v[a];
  }
  for (int sy = 0; sy < 2; ++sy)
    for (int sz = 0; sz < 2; ++sz) {
      const double dy = sy ? 1.0 : -1.0, dz = sz ? 1.0 : -1.0;
      const double my = c.h6[1], mz = c.h6[2], ky = -c.hinv[1], kz = -c.hinv[2];
      c.cyz[sy][sz][0] = my * mz;
      c.cyz[sy][sz][1] = ky * mz + my * kz;
      c.cyz[sy][sz][2] = d.v[1] * 0.5 * dy * mz + d.v[2] * my * 0.5 * dz;
      c.cyz[sy][sz][3] = d.v[0] * my * mz;
    }
  c.ht = 0.5 * d.tau;
  c.inv_tau = 1.0 / d.tau;
  c.tau6 = d.tau / 6.0;
  c.tau3 = d.tau / 3.0;
  c.beta1 = d.beta1;
  c.beta2 = d.beta2;
  c.l2 = d.reg == STKKT_REG_H1L2;
  return c;
}

struct Centre {
  double m, k, c;   // centre mass, stiffness and convection entries of the node on one axis
};

__device__ inline Centre axis_centre(const MvConst &mc, int a, int i, int nn) {
  const bool end = (i == 0) || (i == nn - 1);
  Centre r;
  r.m = end ? 2.0 * mc.h6[a] : 4.0 * mc.h6[a];
  r.k = end ? mc.hinv[a] : 2.0 * mc.hinv[a];
  r.c = (i == 0) ? -0.5 : ((i == nn - 1) ? 0.5 : 0.0);
  return r;
}

// Sums of a node's row over its neighbours: aC, aG (mass) and sC, sG (diffusion
// and convection) of the C and G rows, aF of the f row, from the combined
// fields of the neighbours: at(dy, dz, r) fills r with {U1, S1}, {U2, S2},
// {U3, T3} of the nodes x - 1, x, x + 1 of the line (dy, dz); A[0 .. 26]: the
// node's diffusion entries.
struct RowSums {
  double aC, sC, aG, sG, aF;
};

template <typename Tab, typename At>
__device__ inline RowSums neighbour_sums(const MvConst &mc, const Centre &cx, const Centre &cy, const Centre &cz,
                                         const Tab &A, At at) {
  // Sum factorisation: B, K and N are tensor products of 1-D factors, so
  // each row of three x-neighbours is first contracted with the x factors
  // (off-centre entries are the same for every node, the centre ones are
  // the node's), then weighted by the (y, z) factors of the row.  The
  // variable diffusion A is applied point by point.
  double aC = 0.0, sC = 0.0, aG = 0.0, sG = 0.0, aF = 0.0;
  // The dz planes stay a loop: unrolled, the compiler requests the LDS
  // values of all nine rows at once and their registers leave one
  // wavefront per SIMD.  Rolled, the diffusion table of the node goes to
  // per-lane scratch (cached; 224 B) and two wavefronts fit
  // (174.7 / 642 us against 187.3 / 733 us on cube32x64 / cube48x96).
#pragma unroll 1
  for (int dz = -1; dz <= 1; ++dz) {
#pragma unroll
    for (int dy = -1; dy <= 1; ++dy) {
      double myz, kyz, nyz, vmyz;
      if (dy != 0 && dz != 0) {
        const double *c4 = mc.cyz[dy > 0][dz > 0];
        myz = c4[0];
        kyz = c4[1];
        nyz = c4[2];
        vmyz = c4[3];
      } else if (dy == 0 && dz != 0) {
        myz = cy.m * mc.h6[2];
        kyz = cy.k * mc.h6[2] - cy.m * mc.hinv[2];
        nyz = mc.v[1] * mc.h6[2] * cy.c + (0.5 * dz) * mc.v[2] * cy.m;
        vmyz = mc.v[0] * myz;
      } else if (dy != 0 && dz == 0) {
        myz = mc.h6[1] * cz.m;
        kyz = -mc.hinv[1] * cz.m + mc.h6[1] * cz.k;
        nyz = (0.5 * dy) * mc.v[1] * cz.m + mc.v[2] * mc.h6[1] * cz.c;
        vmyz = mc.v[0] * myz;
      } else {
        myz = cy.m * cz.m;
        kyz = cy.k * cz.m + cy.m * cz.k;
        nyz = mc.v[1] * cy.c * cz.m + mc.v[2] * cy.m * cz.c;
        vmyz = mc.v[0] * myz;
      }
      // N^T differs from N only in the sign of the off-centre convection entries
      double ntyz;
      if (dy != 0 && dz != 0) ntyz = -nyz;
      else if (dy == 0 && dz != 0) ntyz = mc.v[1] * mc.h6[2] * cy.c - (0.5 * dz) * mc.v[2] * cy.m;
      else if (dy != 0 && dz == 0) ntyz = -(0.5 * dy) * mc.v[1] * cz.m + mc.v[2] * mc.h6[1] * cz.c;
      else ntyz = nyz;
      double2 r[9];
      at(dy, dz, r);
      const double2 w1 = r[0], w2 = r[1], w3 = r[2];   // x - 1
      const double2 c1 = r[3], c2 = r[4], c3 = r[5];   // x
      const double2 e1 = r[6], e2 = r[7], e3 = r[8];   // x + 1
      const int k0 = 3 * (dy + 1) + 9 * (dz + 1);
      const double mU1 = mc.h6[0] * (w1.x + e1.x) + cx.m * c1.x;
      const double mU2 = mc.h6[0] * (w2.x + e2.x) + cx.m * c2.x;
      const double mU3 = mc.h6[0] * (w3.x + e3.x) + cx.m * c3.x;
      const double mT = mc.h6[0] * (w3.y + e3.y) + cx.m * c3.y;
      const double kT = cx.k * c3.y - mc.hinv[0] * (w3.y + e3.y);
      const double mS1 = mc.h6[0] * (w1.y + e1.y) + cx.m * c1.y;
      const double cS1 = 0.5 * (e1.y - w1.y) + cx.c * c1.y;
      const double aS1 = A[k0] * w1.y + A[k0 + 1] * c1.y + A[k0 + 2] * e1.y;
      const double mS2 = mc.h6[0] * (w2.y + e2.y) + cx.m * c2.y;
      const double cS2 = 0.5 * (w2.y - e2.y) + cx.c * c2.y;
      const double aS2 = A[k0] * w2.y + A[k0 + 1] * c2.y + A[k0 + 2] * e2.y;
      aC += myz * mU1;
      aG += myz * mU2;
      aF += myz * (mU3 + kT) + kyz * mT;
      sC += aS1 + vmyz * cS1 + nyz * mS1;
      sG += aS2 + vmyz * cS2 + ntyz * mS2;
    }
  }
  return RowSums{aC, sC, aG, sG, aF};
}

}  // namespace stkkt
