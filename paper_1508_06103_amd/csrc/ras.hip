// One-level space-time restricted additive Schwarz with 3x3 point-block
// ILU(0) subdomain solves (Section 3.2 of the paper: overlapping space-time
// decomposition, subdomain matrices taken from F_h on the extended boxes,
// restricted prolongation of the owned part; Section 4: ILU(0)).
//
// Factor storage ("chunk-major SoA"): the rows of a subdomain are grouped by
// wavefront level L = x + 2y + 4z + 8t (every lower neighbour of the 81-point
// stencil has a smaller level) and, inside a level, in 64-row chunks.  For
// every (level, chunk, stencil slot s) with s = (dx+1) + 3(dy+1) + 9(dz+1) +
// 27(dt+1) -- s < 40 the L blocks, s = 40 inv(U_rr), s > 40 the U blocks --
// the blocks of the chunk's rows that have neighbour s inside the box are
// stored entry-major: value(e, k) at off9 + e * cnt + k, k being the rank of
// the row among those rows.  A wavefront of 64 rows reads each entry of a slot
// with one coalesced load, the five slots it owns for a chunk form one
// contiguous stretch, and no padding is stored for neighbours outside the box.
#include <algorithm>
#include <cstdlib>
#include <map>
#include <memory>
#include <tuple>
#include <type_traits>

#include "block33.hpp"
#include "iluk.hpp"
#include "ras.hpp"
#include "stencil.hpp"

namespace stkkt {

namespace {

constexpr int kApplyThreads = 512;
constexpr size_t kRingLdsLimit = 160 * 1024;   // LDS of one gfx950 workgroup
constexpr int kWaves = kApplyThreads / 64;
constexpr int kSlotsPerWave = 40 / kWaves;   // 5
constexpr unsigned kNoNbr = 1023;            // neighbour place of a slot that leaves the box

// A 64-row chunk of a level (device table, read word by word through the scalar cache).
struct ChunkInfo {
  int32_t row0;       // level-order index of its first row
  int32_t rows;       // 1 to 64
  int32_t L, c, R;    // level, index in the level, rows of the level
  int32_t off40;      // factor element of the diagonal group
  int32_t pad_[2];
  int32_t off[2][kWaves];   // of wavefront w's five L (0) or U (1) groups
};
constexpr int kChunkWords = sizeof(ChunkInfo) / 4;
static_assert(kWaves == 8 && kChunkWords == 24, "word offsets 8 + w and 16 + w");

__host__ __device__ inline void slot_off(int s, int &dx, int &dy, int &dz, int &dt) {
  dx = s % 3 - 1;
  dy = (s / 3) % 3 - 1;
  dz = (s / 9) % 3 - 1;
  dt = s / 27 - 1;
}

__host__ __device__ inline bool inside(int x, int y, int z, int t, const int32_t *dims) {
  return x >= 0 && x < dims[0] && y >= 0 && y < dims[1] && z >= 0 && z < dims[2] && t >= 0 && t < dims[3];
}

// The faces through which slot offset (dx, dy, dz, dt) leaves a box: bit k the
// low face of dimension k, bit 4 + k the high one.
__host__ __device__ inline int slot_faces(int dx, int dy, int dz, int dt) {
  return (dx < 0 ? 1 : 0) | (dy < 0 ? 2 : 0) | (dz < 0 ? 4 : 0) | (dt < 0 ? 8 : 0) | (dx > 0 ? 16 : 0) |
         (dy > 0 ? 32 : 0) | (dz > 0 ? 64 : 0) | (dt > 0 ? 128 : 0);
}

__host__ __device__ inline void unpack(uint64_t c, int &x, int &y, int &z, int &t) {
  x = (int)(c & 0xffff);
  y = (int)((c >> 16) & 0xffff);
  z = (int)((c >> 32) & 0xffff);
  t = (int)(c >> 48);
}

// Place of entry e (row-major 3x3) of block k in a group of cnt blocks: the
// entries 0-3 of all blocks as consecutive quads, then entries 4-7 as quads,
// then entry 8.  Groups start on a multiple of kGroupAlign elements, so a
// lane reads its block with two 16-byte loads plus one (FP32) or four plus
// one (FP64).
constexpr int kGroupAlign = 4;

// Most rows a workgroup of factor_lines_kernel factors together (whole x lines),
// and the packed coordinates of an x line.  Line tables exist only for boxes with
// lines of at most kFactorRows nodes and fewer than 1024 nodes on the other axes.
constexpr int kFactorRows = 54;
__host__ __device__ inline int32_t pack_line(int y, int z, int t) { return y | (z << 10) | (t << 20); }
__host__ __device__ inline int64_t blk_pos(int e, int64_t k, int64_t cnt) {
  return e < 4 ? 4 * k + e : e < 8 ? 4 * cnt + 4 * k + (e - 4) : 8 * cnt + k;
}

// Crout-ordered elimination: the entry of row i at slot st is
//   A_it - sum_k L_ik U_kt  over lower neighbours k of i with t an upper
// neighbour of k (slot pair (sk, su) with off(sk) + off(su) = off(st), sk < 40
// < su, sk < st), in ascending k; then L_it = (...) inv(U_tt) for st < 40.
// This is the IKJ ILU(0) of the paper's subdomain solver reordered by entry.
void build_pairs(std::vector<int16_t> &start, std::vector<uint8_t> &pairs) {
  start.assign(82, 0);
  pairs.clear();
  for (int st = 0; st < 81; ++st) {
    start[st] = (int16_t)(pairs.size() / 2);
    int tx, ty, tz, tt;
    slot_off(st, tx, ty, tz, tt);
    for (int sk = 0; sk < 40 && sk < st; ++sk) {
      int kx, ky, kz, kt;
      slot_off(sk, kx, ky, kz, kt);
      const int ux = tx - kx, uy = ty - ky, uz = tz - kz, ut = tt - kt;
      if (ux < -1 || ux > 1 || uy < -1 || uy > 1 || uz < -1 || uz > 1 || ut < -1 || ut > 1) continue;
      const int su = (ux + 1) + 3 * (uy + 1) + 9 * (uz + 1) + 27 * (ut + 1);
      if (su <= 40) continue;
      pairs.push_back((uint8_t)sk);
      pairs.push_back((uint8_t)su);
    }
  }
  start[81] = (int16_t)(pairs.size() / 2);
}

ShapeHost make_shape(const int dims[4]) {
  ShapeHost sh;
  for (int d = 0; d < 4; ++d) sh.dims[d] = dims[d];
  const int lx = dims[0], ly = dims[1], lz = dims[2], lt = dims[3];
  sh.vol = lx * ly * lz * lt;
  sh.nlev = (lx - 1) + 2 * (ly - 1) + 4 * (lz - 1) + 8 * (lt - 1) + 1;
  std::vector<std::vector<uint64_t>> lev(sh.nlev);
  for (int t = 0; t < lt; ++t)
    for (int z = 0; z < lz; ++z)
      for (int y = 0; y < ly; ++y)
        for (int x = 0; x < lx; ++x)
          lev[x + 2 * y + 4 * z + 8 * t].push_back((uint64_t)x | ((uint64_t)y << 16) | ((uint64_t)z << 32) |
                                                   ((uint64_t)t << 48));
  sh.lvl_start.resize(sh.nlev + 1);
  sh.lvl_start[0] = 0;
  for (int L = 0; L < sh.nlev; ++L) {
    sh.lvl_start[L + 1] = sh.lvl_start[L] + (int32_t)lev[L].size();
    sh.rmax = std::max<int>(sh.rmax, (int)lev[L].size());
    for (auto c : lev[L]) sh.coords.push_back(c);
  }
  sh.nchunk = (sh.rmax + 63) / 64;
  // chunk-major factor layout: for level L, 64-row chunk c of the level, slot s,
  // the group of the blocks of the chunk's rows that have neighbour s (block k
  // = rank of its row among them), entry e of block k at ctab.off + blk_pos(e, k, ctab.cnt)
  if ((size_t)sh.nlev * sh.nchunk * 81 * 2 > (size_t)INT32_MAX) throw Error(STKKT_EINVAL, "ras_setup: subdomain too large");
  sh.ctab.assign((size_t)sh.nlev * sh.nchunk * 81 * 2, 0);
  // a row has neighbour s unless it lies on a face through which s leaves the box
  std::vector<uint8_t> code(sh.vol);
  for (int i = 0; i < sh.vol; ++i) {
    int x, y, z, t;
    unpack(sh.coords[i], x, y, z, t);
    code[i] = (uint8_t)((x == 0 ? 1 : 0) | (y == 0 ? 2 : 0) | (z == 0 ? 4 : 0) | (t == 0 ? 8 : 0) |
                        (x == lx - 1 ? 16 : 0) | (y == ly - 1 ? 32 : 0) | (z == lz - 1 ? 64 : 0) |
                        (t == lt - 1 ? 128 : 0));
  }
  uint8_t faces[81];
  for (int s = 0; s < 81; ++s) {
    int dx, dy, dz, dt;
    slot_off(s, dx, dy, dz, dt);
    faces[s] = (uint8_t)slot_faces(dx, dy, dz, dt);
  }
  int64_t off = 0;
  for (int L = 0; L < sh.nlev; ++L) {
    const int r0 = sh.lvl_start[L], R = sh.lvl_start[L + 1] - r0;
    for (int c = 0; c * 64 < R; ++c) {
      const uint8_t *cd = code.data() + r0 + c * 64;
      const int rows = std::min(64, R - c * 64);
      for (int s = 0; s < 81; ++s) {
        const uint8_t fs = faces[s];
        uint8_t n = 0;   // (at most 64: counted in bytes, so that the loop vectorises)
        for (int q = 0; q < rows; ++q) n = (uint8_t)(n + ((cd[q] & fs) == 0));
        const int cnt = n;
        const int64_t len = (9 * (int64_t)cnt + kGroupAlign - 1) / kGroupAlign * kGroupAlign;
        if (off + len > INT32_MAX) throw Error(STKKT_EINVAL, "ras_setup: subdomain too large");
        const size_t i = (((size_t)L * sh.nchunk + c) * 81 + s) * 2;
        sh.ctab[i] = (int32_t)off;
        sh.ctab[i + 1] = cnt;
        off += len;
        sh.nblocks += cnt;
      }
    }
  }
  sh.felems = off;
  // x lines by level y + 2z + 4t (every lower line has a smaller level)
  if (lx <= kFactorRows && ly < 1024 && lz < 1024 && lt < 1024) {
    const int nline = (ly - 1) + 2 * (lz - 1) + 4 * (lt - 1) + 1;
    sh.line_lvl.assign(nline + 1, 0);
    for (int t = 0; t < lt; ++t)
      for (int z = 0; z < lz; ++z)
        for (int y = 0; y < ly; ++y) ++sh.line_lvl[y + 2 * z + 4 * t + 1];
    for (int k = 0; k < nline; ++k) sh.line_lvl[k + 1] += sh.line_lvl[k];
    std::vector<int32_t> at(sh.line_lvl.begin(), sh.line_lvl.end() - 1);
    sh.lines.resize((size_t)ly * lz * lt);
    for (int t = 0; t < lt; ++t)
      for (int z = 0; z < lz; ++z)
        for (int y = 0; y < ly; ++y) sh.lines[at[y + 2 * z + 4 * t]++] = pack_line(y, z, t);
  }
  return sh;
}

// --------------------------------------------------------------------------
// setup: subdomain matrix from the operator formula, then ILU(0), one
// workgroup per subdomain, rows of a level in parallel (one thread per row).
// W holds the subdomain's rows padded to 81 blocks: W[rho][s][e], kWStride
// doubles per row (rows 16-byte aligned).  This form serves preconditioners
// that have a box of more than kFactorRows nodes along x (all their boxes);
// factor_lines_kernel the others.  Both give the same bits.
// --------------------------------------------------------------------------
constexpr int kWStride = 730;

__global__ void __launch_bounds__(256) factor_kernel(OpDev op, const SubInfo *__restrict__ subs,
                                                     const ShapeInfo *__restrict__ shapes,
                                                     const int32_t *__restrict__ lvl_start,
                                                     const uint64_t *__restrict__ coords,
                                                     const int16_t *__restrict__ pstart,
                                                     const uint8_t *__restrict__ pairs, int sub0, double *W,
                                                     int *status) {
  const SubInfo sd = subs[sub0 + blockIdx.x];
  const ShapeInfo sh = shapes[sd.shape];
  const int lx = sh.dims[0], ly = sh.dims[1], lz = sh.dims[2];
  double *Wb = W + sd.wbase;
  for (int L = 0; L < sh.nlev; ++L) {
    const int r0 = lvl_start[sh.lvl_off + L], r1 = lvl_start[sh.lvl_off + L + 1];
    for (int q = r0 + (int)threadIdx.x; q < r1; q += blockDim.x) {
      int x, y, z, t;
      unpack(coords[sh.coord_off + q], x, y, z, t);
      const long long rho = x + (long long)lx * (y + (long long)ly * (z + (long long)lz * t));
      double *Wr = Wb + rho * kWStride;
      const int gx = sd.org[0] + x, gy = sd.org[1] + y, gz = sd.org[2] + z, gn = sd.org[3] + t;
      for (int s = 0; s < 81; ++s) {
        int dx, dy, dz, dt;
        slot_off(s, dx, dy, dz, dt);
        double blk[9];
        if (inside(x + dx, y + dy, z + dz, t + dt, sh.dims)) {
          kkt_block(op, gx, gy, gz, gn, dx, dy, dz, dt, blk);
        } else {
          for (int e = 0; e < 9; ++e) blk[e] = 0.0;
        }
        for (int e = 0; e < 9; ++e) Wr[9 * s + e] = blk[e];
      }
      for (int st = 0; st < 81; ++st) {
        int tx, ty, tz, tt;
        slot_off(st, tx, ty, tz, tt);
        if (!inside(x + tx, y + ty, z + tz, t + tt, sh.dims)) continue;
        double acc[9];
        for (int e = 0; e < 9; ++e) acc[e] = Wr[9 * st + e];
        for (int p = pstart[st]; p < pstart[st + 1]; ++p) {
          const int sk = pairs[2 * p], su = pairs[2 * p + 1];
          int kx, ky, kz, kt;
          slot_off(sk, kx, ky, kz, kt);
          if (!inside(x + kx, y + ky, z + kz, t + kt, sh.dims)) continue;
          const long long rk = rho + kx + (long long)lx * (ky + (long long)ly * (kz + (long long)lz * kt));
          const double *Lik = Wr + 9 * sk;
          const double *Ukt = Wb + rk * kWStride + 9 * su;
          double l[9], u[9];
          for (int e = 0; e < 9; ++e) {
            l[e] = Lik[e];
            u[e] = Ukt[e];
          }
          for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b)
              acc[3 * a + b] -= dot3(l[3 * a], l[3 * a + 1], l[3 * a + 2], u[b], u[3 + b], u[6 + b]);
        }
        if (st < 40) {
          const long long rt = rho + tx + (long long)lx * (ty + (long long)ly * (tz + (long long)lz * tt));
          const double *D = Wb + rt * kWStride + 9 * 40;
          double d[9], o[9];
          for (int e = 0; e < 9; ++e) d[e] = D[e];
          for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b)
              o[3 * a + b] = dot3(acc[3 * a], acc[3 * a + 1], acc[3 * a + 2], d[b], d[3 + b], d[6 + b]);
          for (int e = 0; e < 9; ++e) acc[e] = o[e];
        } else if (st == 40) {
          double o[9];
          bool ok;
          inv33_pivot(acc, o, ok);
          if (!ok) {
            atomicMax(status, 1);
            for (int e = 0; e < 9; ++e) o[e] = 0.0;
          }
          for (int e = 0; e < 9; ++e) acc[e] = o[e];
        }
        for (int e = 0; e < 9; ++e) Wr[9 * st + e] = acc[e];
      }
    }
    __syncthreads();
  }
}

// The same factorisation by x lines.  Row i needs its 39 lower neighbours in
// other lines and then i - 1 in its own; every lower line has a smaller line
// level y + 2z + 4t, and within a line the slots ascend line by line with the
// own line last.  So the rows of a line, and all lines of a level, are taken
// together through the 13 lower lines (dt, dz, dy ascending; three neighbours
// dx = -1, 0, 1 each), and only the last step (i - 1, inversion of the
// diagonal block) runs along x.  Every entry sees the products of the
// sequential IKJ elimination in its order.
//
// One launch takes one line level of every box; a workgroup takes whole lines
// of one box, ROWS rows (27 in four wavefronts, so that two workgroups share a
// compute unit, or 54 in eight).  Nine lanes hold a row: lane q owns the
// targets with (dx, dy) = (q % 3 - 1, q / 3 - 1), nine blocks over (dz, dt), in
// registers.  For one (dy, dz, dt) the blocks U_k and inv(U_kk) of the lower
// lines' rows are copied into LDS, where three rows use each of them, by
// direct loads in two pieces: dt = 0 columns with the diagonal (piece 0) and
// dt = +1 columns (piece 1); the load of one piece overlaps the products of the
// other.  Slots that no row of the line can use (dz outside -1..1) are left out.
//
// What bounds it: the LDS reads (72 B per block product, about 760 a row) and
// the waits between the 26 pieces, which the second workgroup fills; below
// them the U blocks read, 22 KB per row from HBM by the counters (a row's own
// blocks are 6 KB), since a box's window of lines does not fit in L2.  24^3 x 48
// in 108 boxes (1.34 M rows): 19.5 ms on one stream, 16.5 on two; with a thread
// per row, the rows of a point level in parallel, 157 ms.  Preconditioners with a box over 54 nodes
// long keep that form (factor_kernel).
constexpr int kFlUnits0 = 63, kFlUnits1 = 122;   // 16-byte units per row: slots 40..53, 54..80
template <int ROWS> struct FlCfg {
  static constexpr int threads = ROWS > 28 ? 512 : 256;
  // a row's blocks, and its lanes' exchange of one block
  static constexpr size_t lds = (16 * (size_t)(kFlUnits0 + kFlUnits1) + 72) * ROWS;
  static constexpr int max_lines = ROWS / 2;   // (their rows in transit along x fit the blocks' place)
  static_assert(ROWS <= 7 * (threads / 64), "seven rows per wavefront");
  static_assert(lds * (ROWS > 28 ? 1 : 2) <= kRingLdsLimit, "LDS of a compute unit");
  static_assert(sizeof(double) * max_lines * 2 * 9 * 41 <= 16 * (size_t)(kFlUnits0 + kFlUnits1) * ROWS, "rows in transit");
};
static_assert(kFactorRows == 54, "the widest workgroup");

typedef double dbl2u __attribute__((ext_vector_type(2), aligned(8)));

// 3x3 block at p (8-byte aligned)
__device__ inline void ld_blk(const double *p, double (&f)[9]) {
#pragma unroll
  for (int e = 0; e < 9; ++e) f[e] = p[e];
}

__device__ inline void mul_blk(const double (&a)[9], const double (&b)[9], double (&o)[9]) {
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c) o[3 * r + c] = dot3(a[3 * r], a[3 * r + 1], a[3 * r + 2], b[c], b[3 + c], b[6 + c]);
}

__device__ inline void sub_mul_blk(double (&acc)[9], const double (&l)[9], const double (&u)[9]) {
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c)
      acc[3 * r + c] -= dot3(l[3 * r], l[3 * r + 1], l[3 * r + 2], u[c], u[3 + c], u[6 + c]);
}

// one thread's row position in the workgroup and its target column (dx, dy)
struct FlLane {
  int row;        // LDS row: line of the workgroup * lx + x (0 when idle)
  int x, lx;
  int q, tx, ty;
  bool on;        // holds a row
  double *xch;    // the row's nine doubles of exchange space (its lanes are in one wavefront)
};

// block v of lane `from` to the row's nine lanes; all lanes of the wavefront
// take part (lane 63 reads row 6's block)
__device__ inline void fl_share(const FlLane &f, int from, const double (&v)[9], double (&out)[9]) {
  if (f.q == from && f.on) {
#pragma unroll
    for (int e = 0; e < 9; ++e) f.xch[e] = v[e];
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int e = 0; e < 9; ++e) out[e] = f.xch[e];
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
}

// (dz, dt) = (KZ, KT), lower line dy = ky, piece 0: L_ik for dx = -1, 0, 1 and
// the dt = KT targets.
template <int KZ, int KT>
__device__ inline void fl_piece0(const FlLane &f, int ky, bool line_ok, const double *b0, double (&acc)[9][9]) {
  constexpr int jk = (KT + 1) * 3 + KZ + 1;
  const int uy = f.ty - ky;
#pragma unroll 1
  for (int kx = -1; kx <= 1; ++kx) {
    const int qk = (kx + 1) + 3 * (ky + 1);
    const bool ok = f.on && line_ok && f.x + kx >= 0 && f.x + kx < f.lx;
    double a[9], d[9], l[9];
    fl_share(f, qk, acc[jk], a);
    const double *rowk = b0 + (f.row + (ok ? kx : 0)) * (2 * kFlUnits0);
    if (ok) {
      ld_blk(rowk, d);
      mul_blk(a, d, l);
      if (f.q == qk) {
#pragma unroll
        for (int e = 0; e < 9; ++e) acc[jk][e] = l[e];
      }
      const int ux = f.tx - kx;
      if (ux >= -1 && ux <= 1 && uy >= -1 && uy <= 1) {
        const double *uk = rowk + 9 * (ux + 3 * uy);
        double u[9];
        if (uy > 0 || (uy == 0 && ux > 0)) {   // uz = 0: upper columns only
          ld_blk(uk, u);
          sub_mul_blk(acc[jk], l, u);
        }
        if (KZ < 1) {   // uz = 1
          ld_blk(uk + 81, u);
          sub_mul_blk(acc[KZ < 1 ? jk + 1 : jk], l, u);
        }
      }
    }
  }
}

// piece 1: the dt = KT + 1 targets.  b1 holds slots 54.. (KZ >= 0) or the 8
// bytes before slot 63 and slots 63.. (KZ = -1) of every row.
template <int KZ, int KT>
__device__ inline void fl_piece1(const FlLane &f, int ky, bool line_ok, const double *b1, double (&acc)[9][9]) {
  constexpr int jk = (KT + 1) * 3 + KZ + 1;
  const int uy = f.ty - ky;
#pragma unroll 1
  for (int kx = -1; kx <= 1; ++kx) {
    const int qk = (kx + 1) + 3 * (ky + 1);
    const bool ok = f.on && line_ok && f.x + kx >= 0 && f.x + kx < f.lx;
    double l[9];
    fl_share(f, qk, acc[jk], l);
    const int ux = f.tx - kx;
    if (ok && ux >= -1 && ux <= 1 && uy >= -1 && uy <= 1) {
      // block (ux, uy, uz = 0, ut = 1) is slot 67 + ux + 3 uy
      const double *uk = b1 + (f.row + kx) * (2 * kFlUnits1) + 9 * (ux + 3 * uy) + (KZ < 0 ? 1 + 9 * 4 : 9 * 13);
      double u[9];
      if (KZ > -1) {
        ld_blk(uk - 81, u);
        sub_mul_blk(acc[KZ > -1 ? jk + 3 - 1 : jk], l, u);
      }
      ld_blk(uk, u);
      sub_mul_blk(acc[jk + 3], l, u);
      if (KZ < 1) {
        ld_blk(uk + 81, u);
        sub_mul_blk(acc[KZ < 1 ? jk + 3 + 1 : jk], l, u);
      }
    }
  }
}

// Copy units [u0, u0 + nu) (16 bytes each, from the row's start) of the lower
// lines' rows into rows of `stride` units of LDS by direct loads, a wavefront
// writing up to 64 consecutive units of one row at a time.  Lane l of every
// wavefront knows row l of the workgroup: bit l of `has` tells whether the lower
// line exists, `rho` is the row's place in W (there the lower line's row).
// Nothing here waits on memory: the addresses come from lane reads.
template <int THREADS>
__device__ inline void fl_copy(const double *Wb, int rows, int u0, int nu, int stride, double *lds,
                               unsigned long long has, int rho) {
  const int lane = (int)__lane_id();
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  for (int rr = wave; rr < rows; rr += THREADS / 64) {
    if (!((has >> rr) & 1)) continue;
    const double *row = Wb + (long long)__builtin_amdgcn_readlane(rho, rr) * kWStride + 2 * u0;
    double *dst = lds + rr * stride * 2;
    if (lane < nu)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(row + 2 * lane),
                                       (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
    if (lane + 64 < nu)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(row + 128 + 2 * lane),
                                       (__attribute__((address_space(3))) void *)(dst + 128), 16, 0, 0);
  }
}

template <int ROWS>
__global__ void __launch_bounds__(FlCfg<ROWS>::threads, 2) factor_lines_kernel(
    OpDev op, const double *__restrict__ atab, const SubInfo *__restrict__ subs, const ShapeInfo *__restrict__ shapes,
    const int32_t *__restrict__ lines, const int32_t *__restrict__ line_lvl, int sub0, int nsub, int nsub8, int L,
    double *W, int *status) {
  extern __shared__ __align__(16) double fl_lds[];
  constexpr int kThreads = FlCfg<ROWS>::threads;
  // boxes are dealt so that a box stays on one XCD (nsub8 is a multiple of 8)
  const int box = (int)blockIdx.x % nsub8, group = (int)blockIdx.x / nsub8;
  if (box >= nsub) return;
  const SubInfo sd = load_uniform(subs + sub0 + box);
  const ShapeInfo sh = load_uniform(shapes + sd.shape);
  if (L >= sh.nline) return;
  const int lx = sh.dims[0], ly = sh.dims[1], lz = sh.dims[2], lt = sh.dims[3];
  const int per_round = min(ROWS / lx, FlCfg<ROWS>::max_lines);   // lines
  const cptr<int32_t> lvl = as_const(line_lvl) + sh.ll_off;
  const int first = lvl[L] + group * per_round, l1 = lvl[L + 1];
  if (first >= l1) return;
  double *Wb = W + sd.wbase;
  double *b0 = fl_lds, *b1 = fl_lds + (size_t)ROWS * kFlUnits0 * 2;
  const int lane = (int)__lane_id(), wave = (int)(threadIdx.x >> 6);

  FlLane f;
  f.lx = lx;
  const int rw = min(lane / 9, 6);
  f.q = lane - 9 * rw;   // (lane 63: 9, owns nothing)
  f.tx = f.q % 3 - 1;
  f.ty = f.q / 3 - 1;
  const int slot = 7 * wave + rw;
  const int lr = slot / lx;   // line of this row
  f.x = slot - lr * lx;
  const int nl = min(per_round, l1 - first), rows = nl * lx;
  f.on = lane < 63 && lr < nl;
  f.row = f.on ? slot : 0;
  f.xch = fl_lds + (size_t)ROWS * (kFlUnits0 + kFlUnits1) * 2 + 9 * min(slot, ROWS - 1);
  const int32_t pk = lines[sh.ln_off + first + (f.on ? lr : 0)];
  const int y = pk & 1023, z = (pk >> 10) & 1023, t = pk >> 20;
  // lane l: row l of the workgroup, for the copies
  const int cl = lane / lx, cx = lane - cl * lx;
  const int32_t cp = lines[sh.ln_off + first + (cl < nl ? cl : 0)];
  const int cy = cp & 1023, cz = (cp >> 10) & 1023, ct = cp >> 20;
  const int crho = cx + lx * (cy + ly * (cz + lz * ct));
  auto issue = [&](int ky, int kz, int kt, int u0, int nu, int stride, double *lds) {
    const bool in = cl < nl && cy + ky >= 0 && cy + ky < ly && cz + kz >= 0 && cz + kz < lz && ct + kt >= 0;
    fl_copy<kThreads>(Wb, rows, u0, nu, stride, lds, __ballot(in), crho + lx * (ky + ly * (kz + lz * kt)));
  };
  auto issue0 = [&](int ky, int kz, int kt) { issue(ky, kz, kt, 180, kz < 1 ? 63 : 23, kFlUnits0, b0); };
  auto issue1 = [&](int ky, int kz, int kt) {
    issue(ky, kz, kt, kz < 0 ? 283 : 243, kz < 0 ? 82 : kz == 0 ? 122 : 81, kFlUnits1, b1);
  };
  issue0(-1, -1, -1);
  // the rows' blocks of F_h (overlaps the first copy)
  double acc[9][9];
  const int gx = sd.org[0] + f.x, gy = sd.org[1] + y, gz = sd.org[2] + z, gn = sd.org[3] + t;
#pragma unroll
  for (int tz = -1; tz <= 1; ++tz) {
    const bool in3 = f.on && f.x + f.tx >= 0 && f.x + f.tx < lx && y + f.ty >= 0 && y + f.ty < ly && z + tz >= 0 &&
                     z + tz < lz;
    SpatialCoef c{};
    if (in3) {
      const long long node = gx + (long long)op.nn[0] * (gy + (long long)op.nn[1] * gz);
      c = spatial_coef_with(op, gx, gy, gz, f.tx, f.ty, tz, atab[27 * node + f.q + 9 * (tz + 1)]);
    }
#pragma unroll
    for (int tt = -1; tt <= 1; ++tt) {
      const int j = (tt + 1) * 3 + tz + 1;
      if (in3 && t + tt >= 0 && t + tt < lt) {
        kkt_block_c(op, c, gx, gy, gz, gn, f.tx, f.ty, tz, tt, acc[j]);
      } else {
#pragma unroll
        for (int e = 0; e < 9; ++e) acc[j][e] = 0.0;
      }
    }
  }
  auto wait_copies = [] {
    __builtin_amdgcn_s_waitcnt(0);   // the direct loads of this wavefront have reached LDS
    __syncthreads();
  };
  auto line_ok = [&](int ky, int kz, int kt) {
    return y + ky >= 0 && y + ky < ly && z + kz >= 0 && z + kz < lz && t + kt >= 0;
  };
  // the lower lines (dt, dz, dy) ascending; (nky, nkz, nkt): the one after
  auto step = [&](auto KZc, auto KTc, int ky, int nky, int nkz, int nkt, bool last) {
    constexpr int KZ = decltype(KZc)::value, KT = decltype(KTc)::value;
    wait_copies();
    issue1(ky, KZ, KT);
    fl_piece0<KZ, KT>(f, ky, line_ok(ky, KZ, KT), b0, acc);
    wait_copies();
    if (!last) issue0(nky, nkz, nkt);
    fl_piece1<KZ, KT>(f, ky, line_ok(ky, KZ, KT), b1, acc);
  };
  using M1 = std::integral_constant<int, -1>;
  using Z0 = std::integral_constant<int, 0>;
  using P1 = std::integral_constant<int, 1>;
#pragma unroll 1
  for (int ky = -1; ky <= 1; ++ky) step(M1{}, M1{}, ky, ky < 1 ? ky + 1 : -1, ky < 1 ? -1 : 0, -1, false);
#pragma unroll 1
  for (int ky = -1; ky <= 1; ++ky) step(Z0{}, M1{}, ky, ky < 1 ? ky + 1 : -1, ky < 1 ? 0 : 1, -1, false);
#pragma unroll 1
  for (int ky = -1; ky <= 1; ++ky) step(P1{}, M1{}, ky, ky < 1 ? ky + 1 : -1, ky < 1 ? 1 : -1, ky < 1 ? -1 : 0, false);
#pragma unroll 1
  for (int ky = -1; ky <= 1; ++ky) step(M1{}, Z0{}, ky, ky < 1 ? ky + 1 : -1, ky < 1 ? -1 : 0, 0, false);
  step(Z0{}, Z0{}, -1, 0, 0, 0, true);
  // own line, along x: a row's inverse and U blocks pass to the next row
  // through LDS (line's slots 40..80 in piece-0 layout from b0 on, 41
  // blocks per line, two lines' rows alternating by parity of x)
  __syncthreads();
  double *pass = fl_lds + (size_t)(f.on ? lr : 0) * 2 * (9 * 41);
  for (int xs = 0; xs < lx; ++xs) {
    if (f.on && f.x == xs) {
      const double *pv = pass + ((xs + 1) & 1) * (9 * 41);
      double *pw = pass + (xs & 1) * (9 * 41);
      constexpr int jk = 4;   // (dz, dt) = (0, 0)
      if (xs > 0) {
        double a[9], d[9], l[9], u[9];
        const int qk = 3;   // (dx, dy) = (-1, 0)
        fl_share(f, qk, acc[jk], a);
        ld_blk(pv, d);
        mul_blk(a, d, l);
        if (f.q == qk) {
#pragma unroll
          for (int e = 0; e < 9; ++e) acc[jk][e] = l[e];
        }
        const int ux = f.tx + 1, uy = f.ty;
        if (ux <= 1) {
          const double *uk = pv + 9 * (ux + 3 * uy);
          if (uy > 0 || (uy == 0 && ux > 0)) {
            ld_blk(uk, u);
            sub_mul_blk(acc[4], l, u);
          }
          ld_blk(uk + 81, u);
          sub_mul_blk(acc[5], l, u);
          ld_blk(uk + 9 * 18, u);
          sub_mul_blk(acc[6], l, u);
          ld_blk(uk + 9 * 27, u);
          sub_mul_blk(acc[7], l, u);
          ld_blk(uk + 9 * 36, u);
          sub_mul_blk(acc[8], l, u);
        }
      }
      if (f.q == 4) {   // the diagonal block
        double o[9];
        bool ok;
        inv33_pivot(acc[jk], o, ok);
        if (!ok) {
          atomicMax(status, 1);
#pragma unroll
          for (int e = 0; e < 9; ++e) o[e] = 0.0;
        }
#pragma unroll
        for (int e = 0; e < 9; ++e) acc[jk][e] = o[e];
      }
      if (f.q >= 4) {   // slots 40..44
#pragma unroll
        for (int e = 0; e < 9; ++e) pw[9 * (f.q - 4) + e] = acc[jk][e];
      }
#pragma unroll
      for (int j = 5; j < 9; ++j)
#pragma unroll
        for (int e = 0; e < 9; ++e) pw[9 * (f.q + 9 * (j - 4) - 4) + e] = acc[j][e];
    }
    __syncthreads();
  }
  if (f.on) {
    double *Wr = Wb + (f.x + (long long)lx * (y + (long long)ly * (z + (long long)lz * t))) * kWStride + 9 * f.q;
#pragma unroll
    for (int j = 0; j < 9; ++j) {
      double *o = Wr + 81 * j;
#pragma unroll
      for (int e = 0; e < 8; e += 2) *reinterpret_cast<dbl2u *>(o + e) = dbl2u{acc[j][e], acc[j][e + 1]};
      o[8] = acc[j][8];
    }
  }
}

__device__ inline unsigned lanes_below(unsigned long long mask) {
  const unsigned lane = __lane_id();
  return (unsigned)__popcll(mask & ((1ull << lane) - 1ull));
}

// Block `v` into place k of a group of cnt blocks (blk_pos layout, 16-byte aligned quads).
__device__ inline void store_block(double *g, int64_t k, int64_t cnt, const double *v) {
  *reinterpret_cast<double2 *>(g + 4 * k) = make_double2(v[0], v[1]);
  *reinterpret_cast<double2 *>(g + 4 * k + 2) = make_double2(v[2], v[3]);
  *reinterpret_cast<double2 *>(g + 4 * cnt + 4 * k) = make_double2(v[4], v[5]);
  *reinterpret_cast<double2 *>(g + 4 * cnt + 4 * k + 2) = make_double2(v[6], v[7]);
  g[8 * cnt + k] = v[8];
}
__device__ inline void store_block(float *g, int64_t k, int64_t cnt, const double *v) {
  *reinterpret_cast<float4 *>(g + 4 * k) = make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
  *reinterpret_cast<float4 *>(g + 4 * cnt + 4 * k) = make_float4((float)v[4], (float)v[5], (float)v[6], (float)v[7]);
  g[8 * cnt + k] = (float)v[8];
}

// W (rows of 81 blocks) into the chunk-major layout.  A workgroup takes nine
// slots of one 64-row chunk at a time: the rows' 648 bytes come in with
// coalesced reads, on their way while the nine slots before are stored, and are
// turned around in LDS, where lane = row.  Bound by the bytes of W read and F
// written (14 GB at 24^3 x 48 in 108 boxes, 3.1 ms; 5.5 with the loads after the
// stores; 7.1 with one workgroup per box and each lane reading its own row).
// Every box gets kCompactSplit workgroups (its levels in turn).
constexpr int kCompactSplit = 16, kCompactLoads = (64 * 81 + 255) / 256;
template <typename T>
__global__ void __launch_bounds__(256) compact_kernel(const SubInfo *__restrict__ subs,
                                                      const ShapeInfo *__restrict__ shapes,
                                                      const int32_t *__restrict__ lvl_start,
                                                      const uint64_t *__restrict__ coords,
                                                      const int32_t *__restrict__ ctab, int sub0,
                                                      const double *__restrict__ W, T *__restrict__ F) {
  __shared__ double tile[64 * 81];
  __shared__ int32_t rhos[64];
  const SubInfo sd = load_uniform(subs + sub0 + blockIdx.x);
  const ShapeInfo sh = load_uniform(shapes + sd.shape);
  const int lx = sh.dims[0], ly = sh.dims[1], lz = sh.dims[2];
  const int tid = (int)threadIdx.x, lane = (int)__lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const double *Wb = W + sd.wbase;
  for (int L = blockIdx.y; L < sh.nlev; L += gridDim.y) {
    const int r0 = lvl_start[sh.lvl_off + L], R = lvl_start[sh.lvl_off + L + 1] - r0;
    for (int c = 0; c * 64 < R; ++c) {
      const int rows = min(64, R - 64 * c);
      int x = 0, y = 0, z = 0, t = 0;
      if (lane < rows) unpack(coords[sh.coord_off + r0 + 64 * c + lane], x, y, z, t);
      __syncthreads();
      if (wave == 0) rhos[lane] = x + lx * (y + ly * (z + lz * t));
      __syncthreads();   // rhos written
      const int n = rows * 81;
      double pre[kCompactLoads];   // the next nine slots, on their way while the current ones are stored
      auto request = [&](int g) {
#pragma unroll
        for (int i = 0; i < kCompactLoads; ++i) {
          const int q = min(tid + 256 * i, n - 1), rr = q / 81;
          pre[i] = Wb[(long long)rhos[rr] * kWStride + 81 * g + (q - 81 * rr)];
        }
      };
      request(0);
      for (int g = 0; g < 9; ++g) {
        __syncthreads();   // the previous tile read
#pragma unroll
        for (int i = 0; i < kCompactLoads; ++i)
          if (tid + 256 * i < n) tile[tid + 256 * i] = pre[i];
        __syncthreads();
        if (g < 8) request(g + 1);
        for (int j = wave; j < 9; j += 4) {
          const int s = 9 * g + j;
          int dx, dy, dz, dt;
          slot_off(s, dx, dy, dz, dt);
          const bool has = lane < rows && inside(x + dx, y + dy, z + dz, t + dt, sh.dims);
          const unsigned long long mask = __ballot(has);
          // through the scalar cache: a vector load would wait for the requests ahead of it
          const cptr<int32_t> ct = as_const(ctab) + sh.ct_off + (((int64_t)L * sh.nchunk + c) * 81 + s) * 2;
          if (has) {
            store_block(F + sd.fbase + ct[0], (int64_t)lanes_below(mask), (int64_t)ct[1], tile + 81 * lane + 9 * j);
          }
        }
      }
    }
  }
}

// --------------------------------------------------------------------------
// apply: z = sum_i (R^0_i)^T U_i^{-1} L_i^{-1} R^delta_i r
//
// One workgroup (8 wavefronts) per subdomain runs the forward sweep over the
// levels, then the backward sweep.  A level is cut into phases of up to
// kRows rows.  Wavefront w owns 5 of the 40 off-diagonal stencil slots of the
// sweep and walks the 64-row chunks of a phase in "units" of three slots
// (chunk, slots 0-2) and (chunk, slots 3-4): the loads of the next unit
// (factor blocks and neighbour values) are issued before the current unit is
// multiplied, so a wavefront always has a unit of loads in flight.  Partial
// sums go to LDS; after a barrier each thread finishes one row (y = r - sum,
// or z = inv(D)(y - sum)) and a second barrier publishes the new values.
// Everything a phase needs besides the factor stream is requested at the
// start of the phase, ahead of the factor loads: the coordinates of the next
// phase (kept in LDS, so address computation never waits on a vector load)
// and the inputs of the final step (r, or inv(D) and y).
//
// Local vectors use a strided (level, t, z, y) layout
//     row index = L * (lt lz ly) + (t lz + z) ly + y      (x = L - 2y - 4z - 8t)
// so the neighbour of any row through slot s is at a constant offset
// (dx + 2dy + 4dz + 8dt)(lt lz ly) + (dt lz + dz) ly + dy, and the 64 rows of
// a chunk touch nearly contiguous neighbour rows.
// --------------------------------------------------------------------------
constexpr int kRows = 256;
constexpr int kUnit = 3;                     // slots per pipeline unit

template <typename T>
struct SweepArgs {
  SubInfo sd;
  ShapeInfo sh;
  OpDev op;
  cptr<int32_t> lvls;       // shape-relative level starts
  const uint64_t *crd;      // shape coords (read per lane)
  cptr<int32_t> ct;         // shape chunk table: (off9, cnt) per (level, chunk, slot)
  const T *F;
  T *Y;
  int64_t fzero, yzero;
  int64_t SL;               // lt * lz * ly
  const double *r;
  double *z;
};

// (element offset inside the subdomain, count) of the blocks of (level L, chunk cl, slot s).
// All arguments are wavefront-uniform; the index is made so explicitly, so that
// the entry comes through the scalar cache and never queues behind the factor
// loads in flight (a vector load here would have to drain them before the
// addresses that depend on it could be formed).
template <typename T>
__device__ inline void chunk_slot(const SweepArgs<T> &a, int L, int cl, int s, int64_t &off9, int64_t &cnt) {
  const int i = __builtin_amdgcn_readfirstlane(((L * a.sh.nchunk + cl) * 81 + s) * 2);
  off9 = a.ct[i];
  cnt = a.ct[i + 1];
}

// Block k of a group of cnt blocks starting at g (blk_pos layout; g is
// 16-byte aligned): two 16-byte loads and one 4-byte load.
__device__ inline void load_block(const float *g, int64_t k, int64_t cnt, float (&f)[9]) {
  const float4 a = *reinterpret_cast<const float4 *>(g + 4 * k);
  const float4 b = *reinterpret_cast<const float4 *>(g + 4 * cnt + 4 * k);
  f[0] = a.x, f[1] = a.y, f[2] = a.z, f[3] = a.w;
  f[4] = b.x, f[5] = b.y, f[6] = b.z, f[7] = b.w;
  f[8] = g[8 * cnt + k];
}
// FP64: four 16-byte loads and one 8-byte load.
__device__ inline void load_block(const double *g, int64_t k, int64_t cnt, double (&f)[9]) {
  const double2 a = *reinterpret_cast<const double2 *>(g + 4 * k);
  const double2 b = *reinterpret_cast<const double2 *>(g + 4 * k + 2);
  const double2 c = *reinterpret_cast<const double2 *>(g + 4 * cnt + 4 * k);
  const double2 d = *reinterpret_cast<const double2 *>(g + 4 * cnt + 4 * k + 2);
  f[0] = a.x, f[1] = a.y, f[2] = b.x, f[3] = b.y;
  f[4] = c.x, f[5] = c.y, f[6] = d.x, f[7] = d.y;
  f[8] = g[8 * cnt + k];
}

template <typename T>
__device__ inline int64_t yrow_of(const SweepArgs<T> &a, int x, int y, int zc, int t) {
  const int L = x + 2 * y + 4 * zc + 8 * t;
  return (int64_t)L * a.SL + ((int64_t)t * a.sh.dims[2] + zc) * a.sh.dims[1] + y;
}

template <typename T>
__device__ inline int64_t global_row(const SweepArgs<T> &a, int x, int y, int zc, int t) {
  const long long node =
      (a.sd.org[0] + x) + (long long)a.op.nn[0] * ((a.sd.org[1] + y) + (long long)a.op.nn[1] * (a.sd.org[2] + zc));
  return 3 * ((long long)(a.sd.org[3] + t) * a.op.N + node);
}

// Issue the loads of one unit: slots 3h .. 3h+2 of this wavefront's five for
// the lane's row (coordinates cw) in chunk cl of level L.
template <typename T, bool kFwd>
__device__ inline void load_unit(const SweepArgs<T> &a, int L, int cl, bool valid, uint64_t cw, int wave, int h,
                                 T (&f)[kUnit][9], T (&yv)[kUnit][3]) {
  int x, y, zc, t;
  unpack(cw, x, y, zc, t);
  const int64_t own = yrow_of(a, x, y, zc, t);
#pragma unroll
  for (int u = 0; u < kUnit; ++u) {
    const int j = kUnit * h + u;
    const bool real = j < kSlotsPerWave;
    const int s = (kFwd ? 0 : 41) + kSlotsPerWave * wave + (real ? j : 0);
    int dx, dy, dz, dt;
    slot_off(s, dx, dy, dz, dt);
    const bool has = real && valid && inside(x + dx, y + dy, zc + dz, t + dt, a.sh.dims);
    const unsigned long long mask = __ballot(has);
    int64_t off9, cnt;
    chunk_slot(a, L, cl, s, off9, cnt);
    const int64_t dY = (int64_t)(dx + 2 * dy + 4 * dz + 8 * dt) * a.SL + ((int64_t)dt * a.sh.dims[2] + dz) * a.sh.dims[1] + dy;
    // rows without the neighbour read the zero block (k = cnt = 0)
    const int64_t gi = has ? a.sd.fbase + off9 : a.fzero;
    const int64_t k = has ? (int64_t)lanes_below(mask) : 0, kc = has ? cnt : 0;
    const int64_t yi = has ? a.sd.sbase + 3 * (own + dY) : a.yzero;
    load_block(a.F + gi, k, kc, f[u]);
    const T *q = a.Y + yi;
    yv[u][0] = q[0];
    yv[u][1] = q[1];
    yv[u][2] = q[2];
  }
}

template <typename T>
__device__ inline void mac_unit(const T (&f)[kUnit][9], const T (&yv)[kUnit][3], T &a0, T &a1, T &a2) {
#pragma unroll
  for (int u = 0; u < kUnit; ++u) {
    a0 += f[u][0] * yv[u][0] + f[u][1] * yv[u][1] + f[u][2] * yv[u][2];
    a1 += f[u][3] * yv[u][0] + f[u][4] * yv[u][1] + f[u][5] * yv[u][2];
    a2 += f[u][6] * yv[u][0] + f[u][7] * yv[u][1] + f[u][8] * yv[u][2];
  }
}

// Next non-empty level after level counter li of the sweep (-1 if none).
__device__ inline int next_level(cptr<int32_t> lvls, int nlev, int li, bool fwd) {
  for (int k = li + 1; k < nlev; ++k) {
    const int L = fwd ? k : nlev - 1 - k;
    if (lvls[L + 1] > lvls[L]) return k;
  }
  return -1;
}

template <typename T, bool kFwd>
__device__ inline void sweep(const SweepArgs<T> &a, T (*part)[kRows][3], uint64_t *crdL) {
  const int lane = (int)__lane_id();
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int tq = (int)threadIdx.x;
  const int nlev = a.sh.nlev;
  int li = next_level(a.lvls, nlev, -1, kFwd);
  if (li < 0) return;
  // coordinates of the first phase
  {
    const int L = kFwd ? li : nlev - 1 - li;
    const int r0 = a.lvls[L], segR = min(kRows, a.lvls[L + 1] - r0);
    if (tq < segR) crdL[tq] = a.crd[a.sh.coord_off + r0 + tq];
    __syncthreads();
  }
  int seg = 0;
  while (li >= 0) {
    const int L = kFwd ? li : nlev - 1 - li;
    const int r0 = a.lvls[L];
    const int R = a.lvls[L + 1] - r0;
    const int segR = min(kRows, R - seg * kRows);
    const int nch = (segR + 63) >> 6;
    // the phase after this one
    int nli = li, nseg = seg + 1;
    if (nseg * kRows >= R) {
      nli = next_level(a.lvls, nlev, li, kFwd);
      nseg = 0;
    }
    int nsegR = 0, nr0 = 0;
    if (nli >= 0) {
      const int nL = kFwd ? nli : nlev - 1 - nli;
      nr0 = a.lvls[nL];
      nsegR = min(kRows, a.lvls[nL + 1] - nr0 - nseg * kRows);
    }
    // requests issued ahead of the factor stream
    uint64_t cnext = 0;
    if (tq < nsegR) cnext = a.crd[a.sh.coord_off + nr0 + nseg * kRows + tq];
    uint64_t fc = 0;
    T pre[12];
    int64_t gi = 0, yown = 0;
    if (tq < segR) {
      fc = crdL[tq];
      int x, y, zc, t;
      unpack(fc, x, y, zc, t);
      gi = global_row(a, x, y, zc, t);
      yown = a.sd.sbase + 3 * yrow_of(a, x, y, zc, t);
      if (kFwd) {
        pre[0] = (T)a.r[gi];
        pre[1] = (T)a.r[gi + 1];
        pre[2] = (T)a.r[gi + 2];
      } else {
        const int qrow = seg * kRows + tq;   // slot 40: every row of the chunk, rank = row & 63
        int64_t off9, cnt;
        chunk_slot(a, L, __builtin_amdgcn_readfirstlane(qrow >> 6), 40, off9, cnt);
        T dg[9];
        load_block(a.F + a.sd.fbase + off9, qrow & 63, cnt, dg);
#pragma unroll
        for (int e = 0; e < 9; ++e) pre[e] = dg[e];
        pre[9] = a.Y[yown];
        pre[10] = a.Y[yown + 1];
        pre[11] = a.Y[yown + 2];
      }
    }
    // factor stream: units (chunk c, slots 0-2) and (chunk c, slots 3-4)
    const int cl0 = (seg * kRows) >> 6;
    T fA[kUnit][9], yA[kUnit][3], fB[kUnit][9], yB[kUnit][3];
    load_unit<T, kFwd>(a, L, cl0, lane < segR, crdL[lane], wave, 0, fA, yA);
    for (int c = 0; c < nch; ++c) {
      const bool valid = c * 64 + lane < segR;
      const uint64_t cw = crdL[c * 64 + lane];
      load_unit<T, kFwd>(a, L, cl0 + c, valid, cw, wave, 1, fB, yB);
      T a0 = 0, a1 = 0, a2 = 0;
      mac_unit(fA, yA, a0, a1, a2);
      if (c + 1 < nch) {
        const bool valid1 = (c + 1) * 64 + lane < segR;
        load_unit<T, kFwd>(a, L, cl0 + c + 1, valid1, crdL[(c + 1) * 64 + lane], wave, 0, fA, yA);
      }
      mac_unit(fB, yB, a0, a1, a2);
      if (valid) {
        part[wave][c * 64 + lane][0] = a0;
        part[wave][c * 64 + lane][1] = a1;
        part[wave][c * 64 + lane][2] = a2;
      }
    }
    __syncthreads();
    if (tq < segR) {
      T s3[3];
#pragma unroll
      for (int cc = 0; cc < 3; ++cc) {
        T acc = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) acc += part[w][tq][cc];
        s3[cc] = acc;
      }
      T *yr = a.Y + yown;
      if (kFwd) {
        for (int cc = 0; cc < 3; ++cc) yr[cc] = pre[cc] - s3[cc];
      } else {
        T v[3], o[3];
        for (int cc = 0; cc < 3; ++cc) v[cc] = pre[9 + cc] - s3[cc];
        for (int cc = 0; cc < 3; ++cc) o[cc] = pre[3 * cc] * v[0] + pre[3 * cc + 1] * v[1] + pre[3 * cc + 2] * v[2];
        for (int cc = 0; cc < 3; ++cc) yr[cc] = o[cc];
        int x, y, zc, t;
        unpack(fc, x, y, zc, t);
        const SubInfo &sd = a.sd;
        const bool owned = x >= sd.olo[0] && x < sd.ohi[0] && y >= sd.olo[1] && y < sd.ohi[1] && zc >= sd.olo[2] &&
                           zc < sd.ohi[2] && t >= sd.olo[3] && t < sd.ohi[3];
        if (owned)
          for (int cc = 0; cc < 3; ++cc) a.z[gi + cc] = (double)o[cc];
      }
    }
    if (tq < nsegR) crdL[tq] = cnext;
    __syncthreads();
    li = nli;
    seg = nseg;
  }
}

template <typename T>
__global__ void __launch_bounds__(kApplyThreads, 2) apply_kernel(OpDev op, const SubInfo *__restrict__ subs,
                                                                 const int32_t *__restrict__ order,
                                                                 const ShapeInfo *__restrict__ shapes,
                                                                 const int32_t *__restrict__ lvl_start,
                                                                 const uint64_t *__restrict__ coords,
                                                                 const int32_t *__restrict__ ctab,
                                                                 const T *__restrict__ F, T *__restrict__ Y,
                                                                 int64_t fzero, int64_t yzero,
                                                                 const double *__restrict__ r,
                                                                 double *__restrict__ z) {
  __shared__ T part[kWaves][kRows][3];
  __shared__ uint64_t crdL[kRows];
  SweepArgs<T> a;
  const int sub = as_const(order)[blockIdx.x];
  a.sd = load_uniform(subs + sub);
  a.sh = load_uniform(shapes + a.sd.shape);
  a.op = op;
  a.lvls = as_const(lvl_start) + a.sh.lvl_off;
  a.crd = coords;
  a.ct = as_const(ctab) + a.sh.ct_off;
  a.F = F;
  a.Y = Y;
  a.fzero = fzero;
  a.yzero = yzero;
  a.SL = (int64_t)a.sh.dims[3] * a.sh.dims[2] * a.sh.dims[1];
  a.r = r;
  a.z = z;
  sweep<T, true>(a, part, crdL);
  __syncthreads();
  sweep<T, false>(a, part, crdL);
}

// --------------------------------------------------------------------------
// apply, LDS-ring form (used when the ring fits in LDS).
//
// Same split of slots over wavefronts as above, but the values of the last 16
// levels live in an LDS ring (16 is one more than the largest level distance
// between a row and its stencil neighbours, x + 2y + 4z + 8t changes by at most
// 15), so level barriers only synchronise LDS and factor loads stay in flight
// through them: a wavefront streams its factor blocks continuously, DEPTH
// 64-row chunks ahead of the multiply.
//
// Everything that depends on the box shape alone is tabulated, so that a chunk
// costs few instructions besides its loads and products:
//  * ChunkInfo, one entry per chunk in sweep order (scalar loads, one chunk
//    ahead of their use): rows, level, the first factor element of every
//    wavefront's five groups (the groups follow each other, and a group's block
//    count is the number of its rows that have the neighbour);
//  * 8 bytes per (row, wavefront, sweep): for each of the five slots the
//    neighbour's place in its level, kNoNbr if it lies outside the box.  The
//    ring entry, the wavefront's has-neighbour mask and with it the row's rank
//    in the group all follow from it.
// Before the tables every chunk recomputed face tests, (t, z) prefix rows and
// 64-bit addresses, about 500 vector instructions per wavefront against 45
// multiply-adds; the thin levels of small boxes (20 rows) took 3.6 us each.
//
// A sweep walks the chunk list; a phase is up to KR / 64 chunks of one level.
// After a phase's partial sums a barrier, then one thread per row adds the
// eight wavefronts' sums in order, finishes the row, puts it in the ring, and a
// second barrier publishes it.  What that thread needs (r, or inv(U_rr) and y)
// is requested when the phase starts, ahead of the factor loads of the next
// chunk, from coordinates read one phase earlier.  The local vector holds rows
// in level order.  With KR = 64 every chunk is a phase and the loop carries no
// branch, so the compiler's wait counts are exact; boxes whose levels have at
// most 64 rows always take that form.
// --------------------------------------------------------------------------
__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <typename T>
struct RingArgs {
  SubInfo sd;
  int nn0, nn1, N;          // mesh sizes of global_row
  int nchk, rmax, vol;
  cptr<int32_t> ch;         // the shape's chunk list (ChunkInfo words)
  const uint64_t *crd;      // the shape's row coordinates
  const uint2 *nbr;         // the shape's neighbour places
  const T *F;               // the subdomain's factors
  T *Y;                     // its local vector
  const double *r;
  double *z;
};

// One chunk of the sweep for one wavefront (wavefront-uniform).
struct Chk {
  int row0, rows, L, c, R, off;
};

// Chunk i of the sweep order; past the end an entry without rows.
template <typename T, bool kFwd>
__device__ inline Chk chunk_at(const RingArgs<T> &a, int i, int wave) {
  const int k = min(i, a.nchk - 1);
  const cptr<int32_t> e = a.ch + (kFwd ? k : a.nchk - 1 - k) * kChunkWords;
  Chk q{e[0], e[1], e[2], e[3], e[4], e[(kFwd ? 8 : 16) + wave]};
  if (i >= a.nchk) q.rows = 0;
  return q;
}

// PACK = 1: lane = row, the wavefront's five slots one after the other.
// PACK = 2 (levels of at most 32 rows): lanes 32 + i hold row i too and take
// every second slot, so that a chunk needs three groups of loads instead of
// five: the address unit spends 16 cycles on a 16-byte load of a wavefront
// however few of its lanes matter, and at 20 rows a level it was busy two
// thirds of the time.
template <int PACK> constexpr int kSlotRegs = (kSlotsPerWave + PACK - 1) / PACK;
template <int PACK> __device__ inline int lane_row() { return (int)__lane_id() & (64 / PACK - 1); }

// Neighbour places of this lane's row of chunk q.
template <typename T, int PACK>
__device__ inline uint2 load_nbr(const RingArgs<T> &a, const Chk &q, int wave, int dir) {
  const uint2 *p = a.nbr + ((size_t)dir * a.vol + q.row0) * kWaves + wave * q.rows;
  return p[(unsigned)min(lane_row<PACK>(), max(q.rows - 1, 0))];   // masked when used: the load has no branch
}

// Place of the neighbour through the slot this lane holds in register group g (kNoNbr: none).
template <int PACK> __device__ inline unsigned nbr_place(const uint2 &v, int g, bool valid) {
  auto field = [&v](int j) {
    return j >= kSlotsPerWave ? kNoNbr : j < 3 ? (v.x >> (10 * j)) & 1023u : (v.y >> (10 * (j - 3))) & 1023u;
  };
  if (PACK == 1) return valid ? field(g) : kNoNbr;
  const unsigned lo = field(2 * g), hi = field(2 * g + 1);
  return valid ? (__lane_id() < 32 ? lo : hi) : kNoNbr;
}

// 9 elements of a block: quads at byte offsets o and o1, the last element at o2, from a scalar base.
__device__ inline void load_block_at(const double *base, unsigned o, unsigned o1, unsigned o2, double (&f)[9]) {
  const char *p = reinterpret_cast<const char *>(base);
  const double2 a = *reinterpret_cast<const double2 *>(p + o);
  const double2 b = *reinterpret_cast<const double2 *>(p + o + 16);
  const double2 c = *reinterpret_cast<const double2 *>(p + o1);
  const double2 d = *reinterpret_cast<const double2 *>(p + o1 + 16);
  f[0] = a.x, f[1] = a.y, f[2] = b.x, f[3] = b.y;
  f[4] = c.x, f[5] = c.y, f[6] = d.x, f[7] = d.y;
  f[8] = *reinterpret_cast<const double *>(p + o2);
}
__device__ inline void load_block_at(const float *base, unsigned o, unsigned o1, unsigned o2, float (&f)[9]) {
  const char *p = reinterpret_cast<const char *>(base);
  const float4 a = *reinterpret_cast<const float4 *>(p + o);
  const float4 b = *reinterpret_cast<const float4 *>(p + o1);
  f[0] = a.x, f[1] = a.y, f[2] = a.z, f[3] = a.w;
  f[4] = b.x, f[5] = b.y, f[6] = b.z, f[7] = b.w;
  f[8] = *reinterpret_cast<const float *>(p + o2);
}

// Factor loads of register group g of the wavefront's five slots for chunk q:
// 32-bit byte offsets from the first of the five groups; `go` runs through
// them.  Lanes without the neighbour read the block at their rank all the same
// (at most one block past the group, inside the factor buffer); mac_group
// discards it.
template <typename T, int PACK>
__device__ inline void load_group(const RingArgs<T> &a, const Chk &q, const uint2 &nb, int g, unsigned &go, T (&f)[9]) {
  constexpr unsigned kQuad = 4 * sizeof(T);
  const bool valid = lane_row<PACK>() < q.rows;
  const T *base = a.F + q.off;
  auto group_bytes = [](unsigned cnt) {
    return (unsigned)sizeof(T) * ((9 * cnt + kGroupAlign - 1) & ~(unsigned)(kGroupAlign - 1));
  };
  const unsigned long long mask = __ballot(nbr_place<PACK>(nb, g, valid) != kNoNbr);
  const unsigned below = __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
  if (PACK == 1) {
    const unsigned cnt = (unsigned)__popcll(mask);
    load_block_at(base, kQuad * below + go, kQuad * below + (go + kQuad * cnt),
                  (unsigned)sizeof(T) * below + (go + 2 * kQuad * cnt), f);
    go += group_bytes(cnt);
  } else {
    const unsigned c0 = (unsigned)__popc((unsigned)mask), c1 = (unsigned)__popc((unsigned)(mask >> 32));
    const unsigned go1 = go + group_bytes(c0);
    const bool up = __lane_id() >= 32;
    const unsigned k = up ? below - c0 : below;
    const unsigned b0 = up ? go1 : go, b1 = up ? go1 + kQuad * c1 : go + kQuad * c0,
                   b2 = up ? go1 + 2 * kQuad * c1 : go + 2 * kQuad * c0;
    load_block_at(base, kQuad * k + b0, kQuad * k + b1, (unsigned)sizeof(T) * k + b2, f);
    go = go1 + group_bytes(c1);
  }
}

// The value of lane + 32 (in lanes 0..31).
__device__ inline unsigned upper_half(unsigned v) {
  const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return r[1];
}
__device__ inline float upper_half(float v) { return __uint_as_float(upper_half(__float_as_uint(v))); }
__device__ inline double upper_half(double v) {
  return __hiloint2double((int)upper_half((unsigned)__double2hiint(v)), (int)upper_half((unsigned)__double2loint(v)));
}

// Neighbour values of register group g of chunk q from the ring; slot j's
// neighbours lie on level q.L + dl[j].
template <typename T, int PACK>
__device__ inline void ring_values(const RingArgs<T> &a, const Chk &q, const uint2 &nb, const int (&dl)[kSlotsPerWave],
                                   int g, const T *yring, T (&v)[3]) {
  const bool valid = lane_row<PACK>() < q.rows;
  const unsigned pl = min(nbr_place<PACK>(nb, g, valid), (unsigned)(a.rmax - 1));
  auto level = [&](int j) { return ((q.L + dl[min(j, kSlotsPerWave - 1)]) & 15) * (3 * a.rmax); };
  const int lv = PACK == 1 ? level(g) : __lane_id() < 32 ? level(2 * g) : level(2 * g + 1);
  const T *y = yring + lv + 3 * pl;
  v[0] = y[0];
  v[1] = y[1];
  v[2] = y[2];
}

// Products of register group g, added in slot order (lanes below 64 / PACK).
template <typename T, int PACK>
__device__ inline void mac_group(const Chk &q, const uint2 &nb, int g, const T (&f)[9], const T (&u)[3], T &a0, T &a1,
                                 T &a2) {
  const bool valid = lane_row<PACK>() < q.rows;
  const bool has = nbr_place<PACK>(nb, g, valid) != kNoNbr;
  const T t0 = dot3(f[0], f[1], f[2], u[0], u[1], u[2]);
  const T t1 = dot3(f[3], f[4], f[5], u[0], u[1], u[2]);
  const T t2 = dot3(f[6], f[7], f[8], u[0], u[1], u[2]);
  const T s0 = a0 + t0, s1 = a1 + t1, s2 = a2 + t2;
  a0 = has ? s0 : a0;
  a1 = has ? s1 : a1;
  a2 = has ? s2 : a2;
  if (PACK == 2 && 2 * g + 1 < kSlotsPerWave) {
    const bool hup = upper_half(has ? 1u : 0u) != 0;
    const T w0 = a0 + upper_half(t0), w1 = a1 + upper_half(t1), w2 = a2 + upper_half(t2);
    a0 = hup ? w0 : a0;
    a1 = hup ? w1 : a1;
    a2 = hup ? w2 : a2;
  }
}

// A phase as the finishing threads see it: its first chunk in sweep order, the
// thread's row (index in level order, valid if tq < rows) and its coordinates.
struct RingPhase {
  int L, rows;        // level, rows of the phase
  int base;           // level-order index of the phase's first row
  int pos;            // place of that row in its level
  int first, nchk;    // chunks [first, first + nchk) of the sweep
  int off40, cnt40;   // diagonal group of this wavefront's 64 rows of the phase
};

template <typename T, bool kFwd, int KR>
__device__ inline RingPhase phase_from(const RingArgs<T> &a, int i, int wave) {
  constexpr int P = KR / 64;
  const int k = min(i, a.nchk - 1), idx = kFwd ? k : a.nchk - 1 - k;
  const cptr<int32_t> e = a.ch + idx * kChunkWords;
  const int row0 = e[0], c = e[3], R = e[4];
  const int seg = c / P;
  RingPhase p;
  p.L = e[2];
  p.rows = i < a.nchk ? min(KR, R - seg * KR) : 0;
  p.base = row0 - 64 * (c - seg * P);
  p.pos = seg * KR;
  p.first = i;
  p.nchk = (max(p.rows, 1) + 63) >> 6;
  const int w = min(wave, p.nchk - 1);   // this wavefront's chunk of the phase
  p.off40 = a.ch[(idx - c + seg * P + w) * kChunkWords + 5];
  p.cnt40 = min(64, R - 64 * (seg * P + w));
  return p;
}

template <typename T>
__device__ inline int64_t ring_global_row(const RingArgs<T> &a, uint64_t cw) {
  int x, y, zc, t;
  unpack(cw, x, y, zc, t);
  const long long node =
      (a.sd.org[0] + x) + (long long)a.nn0 * ((a.sd.org[1] + y) + (long long)a.nn1 * (a.sd.org[2] + zc));
  return 3 * ((long long)(a.sd.org[3] + t) * a.N + node);
}

// Coordinates of this thread's row of phase p (any row when it has none).
template <typename T> __device__ inline uint64_t phase_crd(const RingArgs<T> &a, const RingPhase &p) {
  return a.crd[p.base + min((int)threadIdx.x, max(p.rows - 1, 0))];
}

// Inputs of the final step of the thread's row: r (forward, kept in FP64 until
// it is used) or inv(U_rr) and y (backward).
template <typename T, bool kFwd>
__device__ inline void load_pre(const RingArgs<T> &a, const RingPhase &p, uint64_t cw, T (&pre)[12],
                                double (&rin)[3]) {
  if (kFwd) {
    const double *r = a.r + ring_global_row(a, cw);
    rin[0] = r[0];
    rin[1] = r[1];
    rin[2] = r[2];
  } else {
    const int tq = min((int)threadIdx.x, max(p.rows - 1, 0));
    T d[9];
    const unsigned k = (unsigned)(tq & 63), cnt = (unsigned)p.cnt40;
    constexpr unsigned kQuad = 4 * sizeof(T);
    load_block_at(a.F + p.off40, kQuad * k, kQuad * k + kQuad * cnt, (unsigned)sizeof(T) * k + 2 * kQuad * cnt, d);
#pragma unroll
    for (int e = 0; e < 9; ++e) pre[e] = d[e];
    const T *y = a.Y + 3 * (int64_t)(p.base + tq);
    pre[9] = y[0];
    pre[10] = y[1];
    pre[11] = y[2];
  }
}

// Final step of a phase, one thread per row: sum the wavefronts' partial
// products, then y = r - sum (forward, y also kept in global memory for the
// backward sweep) or z = inv(U_rr)(y - sum) (backward, owned rows written to
// the output); the result goes into the LDS ring.
template <typename T, bool kFwd, int KR>
__device__ inline void ring_finish(const RingArgs<T> &a, const RingPhase &p, uint64_t cw, T (*part)[KR][3],
                                   const T (&pre)[12], const double (&rin)[3], T *yring) {
  const int tq = (int)threadIdx.x;
  if (tq >= p.rows) return;
  T s3[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    T acc = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) acc += part[w][tq][k];
    s3[k] = acc;
  }
  T o[3];
  if (kFwd) {
    for (int k = 0; k < 3; ++k) o[k] = (T)rin[k] - s3[k];
    T *y = a.Y + 3 * (int64_t)(p.base + tq);
    for (int k = 0; k < 3; ++k) y[k] = o[k];
  } else {
    T v[3];
    for (int k = 0; k < 3; ++k) v[k] = pre[9 + k] - s3[k];
    for (int k = 0; k < 3; ++k) o[k] = dot3(pre[3 * k], pre[3 * k + 1], pre[3 * k + 2], v[0], v[1], v[2]);
    const SubInfo &sd = a.sd;
    int x, y, zc, t;
    unpack(cw, x, y, zc, t);
    const bool owned = x >= sd.olo[0] && x < sd.ohi[0] && y >= sd.olo[1] && y < sd.ohi[1] && zc >= sd.olo[2] &&
                       zc < sd.ohi[2] && t >= sd.olo[3] && t < sd.ohi[3];
    if (owned) {
      double *z = a.z + ring_global_row(a, cw);
      for (int k = 0; k < 3; ++k) z[k] = (double)o[k];
    }
  }
  T *yr = yring + ((p.L & 15) * a.rmax + p.pos + tq) * 3;
  for (int k = 0; k < 3; ++k) yr[k] = o[k];
}

// State of a sweep: chunks i .. i + DEPTH + 1, the neighbour places of chunks
// i .. i + DEPTH, the phase of chunk i and the next.
template <typename T, int DEPTH>
struct RingState {
  int i;
  Chk q[DEPTH + 2];
  uint2 nb[DEPTH + 1];
  RingPhase p, p1;
  uint64_t crd, crd1;
  T pre[12];
  double rin[3];
  int dl[kSlotsPerWave];
};

// One chunk: issue the factor loads of the chunk DEPTH ahead, multiply chunk
// i, and close its phase if it is the phase's last.
template <typename T, bool kFwd, int KR, int PACK, int DEPTH, bool kFinish>
__device__ inline void ring_step(const RingArgs<T> &a, int wave, RingState<T, DEPTH> &s,
                                 const T (&fcur)[kSlotRegs<PACK>][9], T (&fload)[kSlotRegs<PACK>][9],
                                 T (*part)[KR][3], T *yring) {
  constexpr int dir = kFwd ? 0 : 1;
  const int lane = (int)__lane_id();
  if (kFinish && (KR == 64 || s.i == s.p.first)) {
    load_pre<T, kFwd>(a, s.p, s.crd, s.pre, s.rin);
    s.crd1 = phase_crd(a, s.p1);
  }
  const uint2 nbn = load_nbr<T, PACK>(a, s.q[DEPTH + 1], wave, dir);
  const Chk qn = chunk_at<T, kFwd>(a, s.i + DEPTH + 2, wave);
  // loads and products group by group: issued in one go, the chunk's loads
  // would fill the address unit's queue and hold up the products behind them
  T a0 = 0, a1 = 0, a2 = 0;
  T v[2][3];
  ring_values<T, PACK>(a, s.q[0], s.nb[0], s.dl, 0, yring, v[0]);
  unsigned go = 0;
#pragma unroll
  for (int g = 0; g < kSlotRegs<PACK>; ++g) {
    load_group<T, PACK>(a, s.q[DEPTH], s.nb[DEPTH], g, go, fload[g]);
    if (g + 1 < kSlotRegs<PACK>) ring_values<T, PACK>(a, s.q[0], s.nb[0], s.dl, g + 1, yring, v[(g + 1) & 1]);
    mac_group<T, PACK>(s.q[0], s.nb[0], g, fcur[g], v[g & 1], a0, a1, a2);
    __builtin_amdgcn_sched_barrier(0);
  }
  const int prow = (KR == 64 ? 0 : (s.q[0].c % (KR / 64)) * 64) + lane;
  if (lane < s.q[0].rows) {
    part[wave][prow][0] = a0;
    part[wave][prow][1] = a1;
    part[wave][prow][2] = a2;
  }
  ++s.i;
#pragma unroll
  for (int k = 0; k <= DEPTH; ++k) s.q[k] = s.q[k + 1];
  s.q[DEPTH + 1] = qn;
#pragma unroll
  for (int k = 0; k < DEPTH; ++k) s.nb[k] = s.nb[k + 1];
  s.nb[DEPTH] = nbn;
  if (KR == 64 || s.i == s.p.first + s.p.nchk) {
    const RingPhase p2 = phase_from<T, kFwd, KR>(a, s.p1.first + s.p1.nchk, wave);
    lds_barrier();
    if (kFinish) ring_finish<T, kFwd, KR>(a, s.p, s.crd, part, s.pre, s.rin, yring);
    lds_barrier();
    s.p = s.p1;
    s.p1 = p2;
    s.crd = s.crd1;
  }
}

template <typename T, bool kFwd, int KR, int PACK, int DEPTH, bool kFinish>
__device__ inline void sweep_ring(const RingArgs<T> &a, int wave, T (*part)[KR][3], T *yring) {
  constexpr int dir = kFwd ? 0 : 1;
  RingState<T, DEPTH> s;
  s.i = 0;
#pragma unroll
  for (int k = 0; k < DEPTH + 2; ++k) s.q[k] = chunk_at<T, kFwd>(a, k, wave);
#pragma unroll
  for (int k = 0; k < DEPTH + 1; ++k) s.nb[k] = load_nbr<T, PACK>(a, s.q[k], wave, dir);
#pragma unroll
  for (int j = 0; j < kSlotsPerWave; ++j) {
    int dx, dy, dz, dt;
    slot_off((kFwd ? 0 : 41) + kSlotsPerWave * wave + j, dx, dy, dz, dt);
    s.dl[j] = dx + 2 * dy + 4 * dz + 8 * dt;
  }
  s.p = phase_from<T, kFwd, KR>(a, 0, wave);
  s.p1 = phase_from<T, kFwd, KR>(a, s.p.nchk, wave);
  if (kFinish) s.crd = phase_crd(a, s.p);
  T f[DEPTH + 1][kSlotRegs<PACK>][9];
#pragma unroll
  for (int k = 0; k < DEPTH; ++k) {
    unsigned go = 0;
#pragma unroll
    for (int g = 0; g < kSlotRegs<PACK>; ++g) load_group<T, PACK>(a, s.q[k], s.nb[k], g, go, f[k][g]);
  }
  static_assert(DEPTH == 1 || DEPTH == 2, "two or three chunk buffers");
  for (;;) {
    ring_step<T, kFwd, KR, PACK, DEPTH, kFinish>(a, wave, s, f[0], f[DEPTH], part, yring);
    if (s.i >= a.nchk) break;
    ring_step<T, kFwd, KR, PACK, DEPTH, kFinish>(a, wave, s, f[1], f[0], part, yring);
    if (s.i >= a.nchk) break;
    if constexpr (DEPTH == 2) {
      ring_step<T, kFwd, KR, PACK, DEPTH, kFinish>(a, wave, s, f[2], f[1], part, yring);
      if (s.i >= a.nchk) break;
    }
  }
}

// Chunks the factor loads run ahead: two where three chunk buffers fit the registers.
template <typename T, int PACK> constexpr int kDepth = sizeof(T) == 4 || PACK == 2 ? 2 : 1;

// The wavefronts that finish rows and the others run separate copies of the
// loop, so that the others issue none of the finishing threads' loads and both
// have exact wait counts; they meet at the same barriers.
template <typename T, bool kFwd, int KR, int PACK>
__device__ inline void sweep_ring(const RingArgs<T> &a, T (*part)[KR][3], T *yring) {
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (wave < KR / 64) sweep_ring<T, kFwd, KR, PACK, kDepth<T, PACK>, true>(a, wave, part, yring);
  else sweep_ring<T, kFwd, KR, PACK, kDepth<T, PACK>, false>(a, wave, part, yring);
}

// Both sweeps of subdomain `sub` with the values of the last 16 levels in LDS.
template <typename T, int KR, int PACK>
__device__ inline void apply_ring_sub(const OpDev &op, const SubInfo *__restrict__ subs, int sub,
                                      const ShapeInfo *__restrict__ shapes, const uint64_t *__restrict__ coords,
                                      const ChunkInfo *__restrict__ chunks, const uint2 *__restrict__ nbr,
                                      const T *__restrict__ F, T *__restrict__ Y, int rmax,
                                      const double *__restrict__ r, double *__restrict__ z) {
  extern __shared__ __align__(16) unsigned char smem[];
  T(*part)[KR][3] = reinterpret_cast<T(*)[KR][3]>(smem);
  T *yring = reinterpret_cast<T *>(smem + sizeof(T) * kWaves * KR * 3);
  RingArgs<T> a;
  a.sd = load_uniform(subs + sub);
  const ShapeInfo sh = load_uniform(shapes + a.sd.shape);
  a.nn0 = op.nn[0];
  a.nn1 = op.nn[1];
  a.N = op.N;
  a.nchk = sh.nchk;
  a.rmax = rmax;
  a.vol = sh.vol;
  a.ch = reinterpret_cast<cptr<int32_t>>(as_const(chunks + sh.chk_off));
  a.crd = coords + sh.coord_off;
  a.nbr = nbr + sh.nbr_off;
  a.F = F + a.sd.fbase;
  a.Y = Y + a.sd.sbase;
  a.r = r;
  a.z = z;
  sweep_ring<T, true, KR, PACK>(a, part, yring);
  __syncthreads();   // forward results in global memory are read by the backward sweep
  sweep_ring<T, false, KR, PACK>(a, part, yring);
}

template <typename T, int KR, int PACK>
__global__ void __launch_bounds__(kApplyThreads, 2) apply_ring_kernel(
    OpDev op, const SubInfo *__restrict__ subs, const int32_t *__restrict__ order,
    const ShapeInfo *__restrict__ shapes, const uint64_t *__restrict__ coords, const ChunkInfo *__restrict__ chunks,
    const uint2 *__restrict__ nbr, const T *__restrict__ F, T *__restrict__ Y, int rmax, const double *__restrict__ r,
    double *__restrict__ z) {
  const int sub = as_const(order)[blockIdx.x];
  apply_ring_sub<T, KR, PACK>(op, subs, sub, shapes, coords, chunks, nbr, F, Y, rmax, r, z);
}

// One preconditioner of a batched application; its vectors start at element
// voff of the batch's concatenated r and z.
template <typename T>
struct RasBatchDesc {
  OpDev op;
  const SubInfo *subs;
  const ShapeInfo *shapes;
  const uint64_t *coords;
  const ChunkInfo *chunks;
  const uint2 *nbr;
  const T *F;
  T *Y;
  int64_t voff;
  int32_t rmax, pad_;
};

// Work list entry (preconditioner, subdomain), ordered largest box first
// over the whole batch.
template <typename T, int KR, int PACK>
__global__ void __launch_bounds__(kApplyThreads, 2) apply_ring_batch_kernel(const RasBatchDesc<T> *__restrict__ descs,
                                                                            const int2 *__restrict__ work,
                                                                            const int *__restrict__ act,
                                                                            const double *__restrict__ r,
                                                                            const double *__restrict__ r2,
                                                                            double *__restrict__ z) {
  const int2 wk = load_uniform(work + blockIdx.x);
  const int a = as_const(act)[wk.x];
  if (!a) return;
  const RasBatchDesc<T> d = load_uniform(descs + wk.x);
  // The pointers are read as pointers from the constant address space: the
  // compiler then takes them to address global memory and emits global loads.
  // (Pointers rebuilt from copied words would be generic, and generic loads
  // also count against the LDS counter, so every LDS wait of the sweep would
  // drain the factor loads in flight.)
  const cptr<RasBatchDesc<T>> dp = as_const(descs + wk.x);
  apply_ring_sub<T, KR, PACK>(d.op, dp->subs, wk.y, dp->shapes, dp->coords, dp->chunks, dp->nbr, dp->F, dp->Y, d.rmax,
                        (a == 2 ? r2 : r) + d.voff, z + d.voff);
}

// --------------------------------------------------------------------------
// the neighbour places of every shape (setup): rows' places in their levels by
// natural index, then per (sweep, row, wavefront) the five slots' places
// --------------------------------------------------------------------------
__global__ void place_kernel(const ShapeInfo *__restrict__ shapes, const int32_t *__restrict__ lvl_start,
                             const uint64_t *__restrict__ coords, uint16_t *__restrict__ place) {
  const ShapeInfo sh = load_uniform(shapes + blockIdx.y);
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < sh.vol; i += gridDim.x * blockDim.x) {
    int x, y, z, t;
    unpack(coords[sh.coord_off + i], x, y, z, t);
    const int rho = x + sh.dims[0] * (y + sh.dims[1] * (z + sh.dims[2] * t));
    place[sh.coord_off + rho] = (uint16_t)(i - lvl_start[sh.lvl_off + x + 2 * y + 4 * z + 8 * t]);
  }
}

__global__ void nbr_kernel(const ShapeInfo *__restrict__ shapes, const int32_t *__restrict__ lvl_start,
                           const uint64_t *__restrict__ coords, const uint16_t *__restrict__ place,
                           uint2 *__restrict__ nbr) {
  const ShapeInfo sh = load_uniform(shapes + blockIdx.y);
  const int lx = sh.dims[0], ly = sh.dims[1], lz = sh.dims[2];
  for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < 2 * kWaves * sh.vol; q += gridDim.x * blockDim.x) {
    const int i = q / (2 * kWaves), wave = q % kWaves, dir = (q / kWaves) & 1;
    int x, y, z, t;
    unpack(coords[sh.coord_off + i], x, y, z, t);
    const int L = x + 2 * y + 4 * z + 8 * t;
    const int r0 = lvl_start[sh.lvl_off + L], R = lvl_start[sh.lvl_off + L + 1] - r0;
    const int c = (i - r0) >> 6, row0 = r0 + 64 * c, rows = min(64, R - 64 * c);
    unsigned f[kSlotsPerWave];
    for (int j = 0; j < kSlotsPerWave; ++j) {
      int dx, dy, dz, dt;
      slot_off(41 * dir + kSlotsPerWave * wave + j, dx, dy, dz, dt);
      f[j] = inside(x + dx, y + dy, z + dz, t + dt, sh.dims)
                 ? place[sh.coord_off + (x + dx) + lx * ((y + dy) + ly * ((z + dz) + lz * (t + dt)))]
                 : kNoNbr;
    }
    nbr[sh.nbr_off + ((size_t)dir * sh.vol + row0) * kWaves + wave * rows + (i - row0)] =
        make_uint2(f[0] | (f[1] << 10) | (f[2] << 20), f[3] | (f[4] << 10));
  }
}

}  // namespace

// LDS of the ring kernel with KR rows per phase: partial sums and the 16-level value ring.
template <typename T, int KR>
static size_t ring_lds_bytes(const ras *R) {
  return sizeof(T) * kWaves * KR * 3 + sizeof(T) * (size_t)16 * R->ring_rmax * 3;
}

template <typename T, int KR, int PACK>
static void launch_ring(const ras *R, const double *r, double *z, T *Y, hipStream_t s) {
  static bool attr_set = false;
  if (!attr_set) {
    STKKT_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&apply_ring_kernel<T, KR, PACK>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)kRingLdsLimit));
    attr_set = true;
  }
  hipLaunchKernelGGL((apply_ring_kernel<T, KR, PACK>), dim3(R->nsub), dim3(kApplyThreads), (ring_lds_bytes<T, KR>(R)),
                     s, R->d, R->d_subs.as<SubInfo>(), R->d_order.as<int32_t>(), R->d_shapes.as<ShapeInfo>(),
                     R->d_coords.as<uint64_t>(), R->d_chunks.as<ChunkInfo>(), R->d_nbr.as<uint2>(), R->factors.as<T>(),
                     Y, R->ring_rmax, r, z);
}

// Most rows per phase of the ring kernel for this preconditioner: 256 when the
// ring fits with them, else 128 (e.g. 13^4 boxes in FP64), else 64 (14^4 boxes
// in FP64), else 0 (no ring: the kernel with the local vector in global
// memory).  The public query reports it, and the members of a batch share the
// smallest of theirs.  Beside the ring and the partial sums, which are all that
// the kernel keeps, the rule leaves the room that phase coordinates (two or
// three words a row) and the (t, z) groups of 16 levels took in an earlier
// layout: boxes near the lines have been timed with these phases only.
template <typename T>
static int ring_rows(const ras *R) {
  if (R->ring_ltlz > kApplyThreads) return 0;
  const size_t bufs = sizeof(T) == 4 ? 3 : 2, groups = sizeof(int32_t) * (size_t)16 * R->ring_ltlz;
  if (ring_lds_bytes<T, 256>(R) + groups + sizeof(uint64_t) * bufs * 256 <= kRingLdsLimit) return 256;
  if (ring_lds_bytes<T, 128>(R) + groups + sizeof(uint64_t) * bufs * 128 <= kRingLdsLimit) return 128;
  if (ring_lds_bytes<T, 64>(R) + groups + sizeof(uint64_t) * bufs * 64 <= kRingLdsLimit) return 64;
  return 0;
}

// The form that runs, for the given rows per phase and most rows of a level:
// a level of at most 64 rows is one chunk, so phases of 256 rows would be the
// same phases with the branches of longer ones; with at most 32 rows two slots
// share a load (cube8x16, 20 rows a level, FP64: an apply of 335 us against 462
// with one slot a load and 496 with 256 rows; of fatter boxes 64-row phases bring
// little or nothing, 24^3 x 48 FP64 2.03 ms against 1.98 with 256 rows, FP32 1.03
// against 1.05).
struct RingForm {
  int kr, pack;
};
static RingForm ring_form(int rows, int rmax) {
  if (rows >= 64 && rmax <= 32) return {64, 2};
  return {rows > 64 && rmax <= 64 ? 64 : rows, 1};
}

template <typename T>
static void launch_apply(const ras *R, const double *r, double *z, T *Y, hipStream_t s) {
  const RingForm fm = ring_form(ring_rows<T>(R), R->ring_rmax);
  if (fm.pack == 2) {
    launch_ring<T, 64, 2>(R, r, z, Y, s);
  } else if (fm.kr == 256) {
    launch_ring<T, 256, 1>(R, r, z, Y, s);
  } else if (fm.kr == 128) {
    launch_ring<T, 128, 1>(R, r, z, Y, s);
  } else if (fm.kr == 64) {
    launch_ring<T, 64, 1>(R, r, z, Y, s);
  } else {
    hipLaunchKernelGGL((apply_kernel<T>), dim3(R->nsub), dim3(kApplyThreads), 0, s, R->d, R->d_subs.as<SubInfo>(),
                       R->d_order.as<int32_t>(), R->d_shapes.as<ShapeInfo>(), R->d_lvl.as<int32_t>(),
                       R->d_coords.as<uint64_t>(), R->d_ctab.as<int32_t>(), R->factors.as<T>(), Y,
                       R->factor_elems, R->scratch_elems, r, z);
  }
}

size_t ras_local_bytes(const ras *R) {
  if (R->iluk) return iluk_local_bytes(R);
  const size_t esz = R->params.precision == STKKT_F32 ? sizeof(float) : sizeof(double);
  return esz * ((size_t)R->scratch_elems + 4);
}

bool ras_uses_ring(const ras *R) {
  if (R->iluk) return false;
  return (R->params.precision == STKKT_F32 ? ring_rows<float>(R) : ring_rows<double>(R)) == 256;
}

int ras_apply_rows_per_phase(const ras *R) {
  if (R->iluk) return 0;
  return R->params.precision == STKKT_F32 ? ring_rows<float>(R) : ring_rows<double>(R);
}

void ras_apply_device(const ras *R, const double *r, double *z, hipStream_t s, void *local) {
  if (R->iluk) {
    iluk_apply(R, r, z, local, s);
    return;
  }
  if (R->params.precision == STKKT_F32)
    launch_apply<float>(R, r, z, local ? static_cast<float *>(local) : R->scratch.as<float>(), s);
  else
    launch_apply<double>(R, r, z, local ? static_cast<double *>(local) : R->scratch.as<double>(), s);
  STKKT_HIP(hipGetLastError());
}

template <typename T>
static void ras_batch_prepare_t(const ras *const *R, const long long *voff, void *const *local, int count,
                                const std::vector<char> &solo, const Allocator *al, RasBatch &out, hipStream_t s) {
  std::vector<RasBatchDesc<T>> d(count);
  std::vector<std::pair<int64_t, int2>> items;
  size_t lds = 0;
  for (int i = 0; i < count; ++i) {
    const ras *q = R[i];
    d[i] = RasBatchDesc<T>{};
    if (!q || solo[i]) continue;   // empty slot, or launched on its own
    d[i].op = q->d;
    d[i].subs = q->d_subs.as<SubInfo>();
    d[i].shapes = q->d_shapes.as<ShapeInfo>();
    d[i].coords = q->d_coords.as<uint64_t>();
    d[i].chunks = q->d_chunks.as<ChunkInfo>();
    d[i].nbr = q->d_nbr.as<uint2>();
    d[i].F = q->factors.as<T>();
    d[i].Y = local && local[i] ? static_cast<T *>(local[i]) : q->scratch.as<T>();
    d[i].voff = voff[i];
    d[i].rmax = q->ring_rmax;
    lds = std::max(lds, out.kr == 256   ? ring_lds_bytes<T, 256>(q)
                        : out.kr == 128 ? ring_lds_bytes<T, 128>(q)
                                        : ring_lds_bytes<T, 64>(q));
    for (int k = 0; k < q->nsub; ++k)
      items.push_back({q->shapes[q->subs[k].shape].nblocks, make_int2(i, k)});
  }
  std::stable_sort(items.begin(), items.end(), [](const auto &a, const auto &b) { return a.first > b.first; });
  std::vector<int2> work(items.size());
  for (size_t k = 0; k < items.size(); ++k) work[k] = items[k].second;
  out.desc = DevBuf(al, sizeof(RasBatchDesc<T>) * (size_t)count);
  out.work = DevBuf(al, sizeof(int2) * std::max<size_t>(work.size(), 1));
  STKKT_HIP(hipMemcpyAsync(out.desc.ptr, d.data(), sizeof(RasBatchDesc<T>) * (size_t)count, hipMemcpyHostToDevice, s));
  STKKT_HIP(hipMemcpyAsync(out.work.ptr, work.data(), sizeof(int2) * work.size(), hipMemcpyHostToDevice, s));
  STKKT_HIP(hipStreamSynchronize(s));   // host staging is released on return
  out.blocks = (int)work.size();
  out.lds = lds;
}

// One launch covers every member whose LDS ring fits, with the largest rows
// per phase (256, 128 or 64) that all of them allow (the per-row sums, and
// so the results, are the same for every phase size and form).  Members without a ring (or with ILU(k) factors)
// are launched on their own after it; members of different precisions make
// every member its own launch.
void ras_batch_prepare(const ras *const *R, const long long *voff, void *const *local, int count,
                       const Allocator *al, RasBatch &out, hipStream_t s) {
  out = RasBatch{};
  out.count = count;
  out.precision = -1;
  bool uniform = true;
  for (int i = 0; i < count; ++i) {
    out.members.push_back(R[i]);
    out.voff.push_back(voff[i]);
    out.local.push_back(local ? local[i] : nullptr);
    if (!R[i]) continue;
    if (out.precision < 0) out.precision = R[i]->params.precision;
    uniform = uniform && R[i]->params.precision == out.precision;
  }
  if (out.precision < 0) out.precision = STKKT_F64;
  if (!uniform) return;   // per-preconditioner launches
  std::vector<char> solo(count, 0);
  int kr = 256, rmax = 0;
  bool any = false;
  for (int i = 0; i < count; ++i) {
    if (!R[i]) continue;
    const int rows = ras_apply_rows_per_phase(R[i]);   // 256, 128, 64, or 0 (no ring, ILU(k))
    if (rows == 0) {
      solo[i] = 1;
      out.solo.push_back(i);
    } else {
      any = true;
      kr = std::min(kr, rows);
      rmax = std::max(rmax, R[i]->ring_rmax);
    }
  }
  if (!any) {   // every member on its own
    out.solo.clear();
    return;
  }
  out.ring = true;
  out.kr = ring_form(kr, rmax).kr;
  out.pack = ring_form(kr, rmax).pack;
  if (out.precision == STKKT_F32) ras_batch_prepare_t<float>(R, voff, local, count, solo, al, out, s);
  else ras_batch_prepare_t<double>(R, voff, local, count, solo, al, out, s);
}

template <typename T, int KR, int PACK>
static void ras_batch_launch_form(const RasBatch &b, const double *r, const double *r2, double *z, const int *act,
                                  hipStream_t s) {
  static bool attr_set = false;
  if (!attr_set) {
    STKKT_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&apply_ring_batch_kernel<T, KR, PACK>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)kRingLdsLimit));
    attr_set = true;
  }
  hipLaunchKernelGGL((apply_ring_batch_kernel<T, KR, PACK>), dim3(b.blocks), dim3(kApplyThreads), b.lds, s,
                     b.desc.as<RasBatchDesc<T>>(), b.work.as<int2>(), act, r, r2 ? r2 : r, z);
}

template <typename T>
static void ras_batch_launch(const RasBatch &b, const double *r, const double *r2, double *z, const int *act,
                             hipStream_t s) {
  if (b.pack == 2) ras_batch_launch_form<T, 64, 2>(b, r, r2, z, act, s);
  else if (b.kr == 256) ras_batch_launch_form<T, 256, 1>(b, r, r2, z, act, s);
  else if (b.kr == 128) ras_batch_launch_form<T, 128, 1>(b, r, r2, z, act, s);
  else ras_batch_launch_form<T, 64, 1>(b, r, r2, z, act, s);
}

void ras_batch_run(const RasBatch &b, const double *r, double *z, const int *act, const int *act_host,
                   hipStream_t s, const double *r2) {
  if (!b.ring) {
    for (int i = 0; i < b.count; ++i)
      if (act_host[i] && b.members[i])
        ras_apply_device(b.members[i], (act_host[i] == 2 && r2 ? r2 : r) + b.voff[i], z + b.voff[i], s,
                         b.local[i]);
    return;
  }
  if (b.blocks > 0) {
    if (b.precision == STKKT_F32) ras_batch_launch<float>(b, r, r2, z, act, s);
    else ras_batch_launch<double>(b, r, r2, z, act, s);
    STKKT_HIP(hipGetLastError());
  }
  for (const int i : b.solo)
    if (act_host[i])
      ras_apply_device(b.members[i], (act_host[i] == 2 && r2 ? r2 : r) + b.voff[i], z + b.voff[i], s, b.local[i]);
}

static std::vector<int> split(int L, int p) {
  std::vector<int> s(p + 1);
  const int q = L / p, r = L % p;
  for (int k = 0; k <= p; ++k) s[k] = k * q + std::min(k, r);
  return s;
}

template <class V> static void upload(const Allocator *al, DevBuf &buf, const std::vector<V> &host, hipStream_t s) {
  buf = DevBuf(al, std::max<size_t>(sizeof(V) * host.size(), 256));
  if (!host.empty())
    STKKT_HIP(hipMemcpyAsync(buf.ptr, host.data(), sizeof(V) * host.size(), hipMemcpyHostToDevice, s));
}

// The chunk list of a shape, in forward sweep order.
static void append_chunks(const ShapeHost &sh, std::vector<ChunkInfo> &out) {
  for (int L = 0; L < sh.nlev; ++L) {
    const int r0 = sh.lvl_start[L], R = sh.lvl_start[L + 1] - r0;
    for (int c = 0; c * 64 < R; ++c) {
      const int32_t *ct = sh.ctab.data() + ((size_t)L * sh.nchunk + c) * 81 * 2;
      ChunkInfo q{};
      q.row0 = r0 + 64 * c;
      q.rows = std::min(64, R - 64 * c);
      q.L = L;
      q.c = c;
      q.R = R;
      q.off40 = ct[2 * 40];
      for (int w = 0; w < kWaves; ++w) {
        q.off[0][w] = ct[2 * (kSlotsPerWave * w)];
        q.off[1][w] = ct[2 * (41 + kSlotsPerWave * w)];
      }
      out.push_back(q);
    }
  }
}

// A second stream of default priority that starts where s stands; join() lets s
// wait for it.  The destructor waits for what it was given.
struct SideStream {
  hipStream_t stream = nullptr;
  hipEvent_t event = nullptr;
  explicit SideStream(hipStream_t s) {
    try {
      STKKT_HIP(hipStreamCreateWithFlags(&stream, hipStreamNonBlocking));
      STKKT_HIP(hipEventCreateWithFlags(&event, hipEventDisableTiming));
      STKKT_HIP(hipEventRecord(event, s));
      STKKT_HIP(hipStreamWaitEvent(stream, event, 0));
    } catch (...) {
      release();
      throw;
    }
  }
  ~SideStream() { release(); }
  void join(hipStream_t s) {
    STKKT_HIP(hipEventRecord(event, stream));
    STKKT_HIP(hipStreamWaitEvent(s, event, 0));
  }
  void release() {
    if (stream) (void)hipStreamSynchronize(stream);
    if (event) (void)hipEventDestroy(event);
    if (stream) (void)hipStreamDestroy(stream);
    event = nullptr;
    stream = nullptr;
  }
  SideStream(const SideStream &) = delete;
  SideStream &operator=(const SideStream &) = delete;
};

constexpr int kFlTwoStreams = 32;   // boxes

template <int ROWS>
static void factor_by_lines_t(const ras *R, const double *atab, const int32_t *lines, const int32_t *line_lvl, int first,
                              int last, double *W, int *status, hipStream_t s) {
  STKKT_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&factor_lines_kernel<ROWS>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)FlCfg<ROWS>::lds));
  // most workgroups any of the boxes has at a line level
  std::vector<char> used(R->shapes.size(), 0);
  for (int i = first; i < last; ++i) used[R->subs[i].shape] = 1;
  std::vector<int> groups;
  for (size_t k = 0; k < R->shapes.size(); ++k) {
    if (!used[k]) continue;
    const ShapeHost &sh = R->shapes[k];
    const int per = std::min(ROWS / sh.dims[0], FlCfg<ROWS>::max_lines), nline = (int)sh.line_lvl.size() - 1;
    if ((int)groups.size() < nline) groups.resize(nline, 0);
    for (int L = 0; L < nline; ++L)
      groups[L] = std::max(groups[L], (sh.line_lvl[L + 1] - sh.line_lvl[L] + per - 1) / per);
  }
  // Boxes are independent: two halves on two streams fill the compute units
  // that a launch's last workgroups leave idle (ras_setup in FP64: 108 boxes of
  // 24^3 x 48 25.0 -> 21.7 ms, 512 of 32^3 x 64 69.1 -> 65.5, 32 of 24^3 x 16
  // 17.0 -> 15.3; fewer leave compute units idle in any case).
  const int mid = last - first >= kFlTwoStreams ? first + (last - first) / 2 : last;
  auto level = [&](int L, int b0, int b1, hipStream_t st) {
    const int count = b1 - b0, count8 = (count + 7) / 8 * 8;
    hipLaunchKernelGGL(factor_lines_kernel<ROWS>, dim3((unsigned)count8 * groups[L]), dim3(FlCfg<ROWS>::threads),
                       FlCfg<ROWS>::lds, st, R->d, atab, R->d_subs.as<SubInfo>(), R->d_shapes.as<ShapeInfo>(), lines,
                       line_lvl, b0, count, count8, L, W, status);
  };
  std::unique_ptr<SideStream> side;
  if (mid < last) side = std::make_unique<SideStream>(s);
  for (int L = 0; L < (int)groups.size(); ++L) {
    if (groups[L] == 0) continue;
    level(L, first, mid, s);
    if (side) level(L, mid, last, side->stream);
  }
  if (side) side->join(s);
}

// Factor the boxes [first, last) line level by line level.  27 rows per
// workgroup (two workgroups per compute unit) unless 54 fill their places
// better: whole x lines are taken, and a line may not fit in 27.
static void factor_by_lines(const ras *R, const double *atab, const int32_t *lines, const int32_t *line_lvl, int first,
                            int last, double *W, int *status, hipStream_t s) {
  long long full27 = 0, full54 = 0;   // rows of full workgroups, in 54ths
  bool fits27 = true;
  for (int i = first; i < last; ++i) {
    const int lx = R->shapes[R->subs[i].shape].dims[0];
    fits27 = fits27 && lx <= 27;
    full27 += 2 * (27 / lx) * lx;
    full54 += (54 / lx) * lx;
  }
  if (fits27 && full27 >= full54 * 4 / 5) factor_by_lines_t<27>(R, atab, lines, line_lvl, first, last, W, status, s);
  else factor_by_lines_t<54>(R, atab, lines, line_lvl, first, last, W, status, s);
}

ras *ras_create(const kkt_op *op, const ras_params_t *rp, hipStream_t s) {
  STKKT_REQUIRE(rp != nullptr, "ras_setup: params is NULL");
  STKKT_REQUIRE(rp->ilu_level >= 0 && rp->ilu_level <= 3, "ras_setup: ilu_level must be 0, 1, 2 or 3");
  STKKT_REQUIRE(rp->precision == STKKT_F64 || rp->precision == STKKT_F32, "ras_setup: bad precision");
  STKKT_REQUIRE(rp->overlap >= 0, "ras_setup: negative overlap");
  const int L[4] = {op->d.nn[0], op->d.nn[1], op->d.nn[2], op->d.M + 1};
  for (int d = 0; d < 4; ++d)
    STKKT_REQUIRE(rp->p[d] >= 1 && rp->p[d] <= L[d], "ras_setup: parts must be in [1, nodes] per dimension");
  auto R = std::make_unique<ras>();
  R->op = op;
  R->al = op->al;
  R->d = op->d;
  R->params = *rp;
  std::vector<int> cut[4];
  for (int d = 0; d < 4; ++d) cut[d] = split(L[d], rp->p[d]);
  const int nsub = rp->p[0] * rp->p[1] * rp->p[2] * rp->p[3];
  R->nsub = nsub;
  std::map<std::tuple<int, int, int, int>, int> shape_id;
  int64_t fb = 0, sb = 0;
  for (int kt = 0; kt < rp->p[3]; ++kt)
    for (int kz = 0; kz < rp->p[2]; ++kz)
      for (int ky = 0; ky < rp->p[1]; ++ky)
        for (int kx = 0; kx < rp->p[0]; ++kx) {
          const int k[4] = {kx, ky, kz, kt};
          int lo[4], hi[4], blo[4], bhi[4], dims[4];
          for (int d = 0; d < 4; ++d) {
            lo[d] = cut[d][k[d]];
            hi[d] = cut[d][k[d] + 1];
            blo[d] = std::max(0, lo[d] - rp->overlap);
            bhi[d] = std::min(L[d], hi[d] + rp->overlap);
            dims[d] = bhi[d] - blo[d];
            STKKT_REQUIRE(dims[d] < 65536, "ras_setup: box too large");
          }
          auto key = std::make_tuple(dims[0], dims[1], dims[2], dims[3]);
          auto it = shape_id.find(key);
          int sid;
          if (it == shape_id.end()) {
            sid = (int)R->shapes.size();
            shape_id[key] = sid;
            R->shapes.push_back(make_shape(dims));
          } else {
            sid = it->second;
          }
          SubInfo si{};
          si.shape = sid;
          for (int d = 0; d < 4; ++d) {
            si.org[d] = blo[d];
            si.olo[d] = lo[d] - blo[d];
            si.ohi[d] = hi[d] - blo[d];
          }
          const ShapeHost &sh = R->shapes[sid];
          si.fbase = fb;
          si.sbase = sb;
          fb += sh.felems;
          R->total_blocks += sh.nblocks;
          sb += 3LL * sh.nlev * sh.dims[3] * sh.dims[2] * sh.dims[1];
          R->subs.push_back(si);
          for (int d = 0; d < 4; ++d) {
            R->boxes.push_back(lo[d]);
          }
          for (int d = 0; d < 4; ++d) R->boxes.push_back(hi[d]);
          for (int d = 0; d < 4; ++d) R->boxes.push_back(blo[d]);
          for (int d = 0; d < 4; ++d) R->boxes.push_back(bhi[d]);
        }
  R->factor_elems = fb;
  R->scratch_elems = sb;
  if (rp->ilu_level > 0) {   // ILU(k): its own pattern, layout and kernels
    R->total_blocks = 0;
    iluk_create(R.get(), op, s);
    return R.release();
  }
  // launch order: largest boxes first, so that the last workgroups to start are the short ones
  std::vector<int32_t> order(nsub);
  for (int i = 0; i < nsub; ++i) order[i] = i;
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
    return R->shapes[R->subs[a].shape].nblocks > R->shapes[R->subs[b].shape].nblocks;
  });
  // shape tables
  std::vector<ShapeInfo> shinfo;
  std::vector<int32_t> lvl;
  std::vector<uint64_t> crd;
  std::vector<int32_t> ctb;
  std::vector<ChunkInfo> chunks;
  int64_t nbr_rows = 0;
  std::vector<int32_t> lines, line_lvl;
  bool by_lines = true;   // every box has line tables
  for (auto &sh : R->shapes) {
    ShapeInfo si{};
    for (int d = 0; d < 4; ++d) si.dims[d] = sh.dims[d];
    si.nlev = sh.nlev;
    si.nchunk = sh.nchunk;
    si.rmax = sh.rmax;
    si.vol = sh.vol;
    si.lvl_off = (int64_t)lvl.size();
    si.coord_off = (int64_t)crd.size();
    si.ct_off = (int64_t)ctb.size();
    si.chk_off = (int64_t)chunks.size();
    si.nbr_off = 2 * kWaves * nbr_rows;
    nbr_rows += sh.vol;
    append_chunks(sh, chunks);
    si.nchk = (int32_t)((int64_t)chunks.size() - si.chk_off);
    si.ln_off = (int64_t)lines.size();
    si.ll_off = (int64_t)line_lvl.size();
    si.nline = (int32_t)sh.line_lvl.size() - 1;
    by_lines = by_lines && !sh.lines.empty();
    R->ring_rmax = std::max(R->ring_rmax, sh.rmax);
    R->ring_ltlz = std::max(R->ring_ltlz, sh.dims[3] * sh.dims[2]);
    lvl.insert(lvl.end(), sh.lvl_start.begin(), sh.lvl_start.end());
    crd.insert(crd.end(), sh.coords.begin(), sh.coords.end());
    ctb.insert(ctb.end(), sh.ctab.begin(), sh.ctab.end());
    lines.insert(lines.end(), sh.lines.begin(), sh.lines.end());
    line_lvl.insert(line_lvl.end(), sh.line_lvl.begin(), sh.line_lvl.end());
    shinfo.push_back(si);
  }
  const Allocator *al = &R->al;
  upload(al, R->d_shapes, shinfo, s);
  upload(al, R->d_lvl, lvl, s);
  upload(al, R->d_coords, crd, s);
  upload(al, R->d_ctab, ctb, s);
  upload(al, R->d_chunks, chunks, s);
  R->d_nbr = DevBuf(al, sizeof(uint2) * 2 * kWaves * (size_t)nbr_rows);
  DevBuf d_place(al, sizeof(uint16_t) * (size_t)nbr_rows);
  {
    const dim3 g(blocks_for(nbr_rows / (int64_t)R->shapes.size() + 1, 256, 256), (unsigned)R->shapes.size());
    hipLaunchKernelGGL(place_kernel, g, dim3(256), 0, s, R->d_shapes.as<ShapeInfo>(), R->d_lvl.as<int32_t>(),
                       R->d_coords.as<uint64_t>(), d_place.as<uint16_t>());
    hipLaunchKernelGGL(nbr_kernel, dim3(8 * g.x, g.y), dim3(256), 0, s, R->d_shapes.as<ShapeInfo>(),
                       R->d_lvl.as<int32_t>(), R->d_coords.as<uint64_t>(), d_place.as<uint16_t>(),
                       R->d_nbr.as<uint2>());
    STKKT_HIP(hipGetLastError());
  }
  upload(al, R->d_order, order, s);
  std::vector<int16_t> pstart;
  std::vector<uint8_t> pairs;
  build_pairs(pstart, pairs);
  DevBuf d_pstart, d_pairs, d_lines, d_line_lvl;
  upload(al, d_pstart, pstart, s);
  upload(al, d_pairs, pairs, s);
  upload(al, d_lines, lines, s);
  upload(al, d_line_lvl, line_lvl, s);
  const size_t esz = rp->precision == STKKT_F32 ? sizeof(float) : sizeof(double);
  // trailing all-zero sentinels read for neighbours outside a box
  R->factors = DevBuf(al, esz * ((size_t)fb + 16));
  R->scratch = DevBuf(al, esz * ((size_t)sb + 4));
  STKKT_HIP(hipMemsetAsync(static_cast<char *>(R->factors.ptr) + esz * (size_t)fb, 0, esz * 16, s));
  STKKT_HIP(hipMemsetAsync(static_cast<char *>(R->scratch.ptr) + esz * (size_t)sb, 0, esz * 4, s));
  // working buffer: subdomains factored in batches that fit the budget
  size_t budget = (size_t)64 << 30;
  if (const char *e = getenv("STKKT_SETUP_WORK_GB")) budget = (size_t)(atof(e) * (double)(1ull << 30));
  size_t free_b = 0, total_b = 0;
  if (hipMemGetInfo(&free_b, &total_b) == hipSuccess && free_b > 0) budget = std::min(budget, free_b / 2);
  DevBuf d_status(al, 256);
  STKKT_HIP(hipMemsetAsync(d_status.ptr, 0, sizeof(int), s));
  int first = 0;
  while (first < nsub) {
    size_t used = 0;
    int last = first;
    while (last < nsub) {
      const size_t need = (size_t)R->shapes[R->subs[last].shape].vol * kWStride * sizeof(double);
      if (last > first && used + need > budget) break;
      R->subs[last].wbase = (int64_t)(used / sizeof(double));
      used += need;
      ++last;
    }
    if (first == 0) upload(al, R->d_subs, R->subs, s);
    else STKKT_HIP(hipMemcpyAsync(R->d_subs.ptr, R->subs.data(), sizeof(SubInfo) * R->subs.size(),
                                  hipMemcpyHostToDevice, s));
    DevBuf work(al, used);
    STKKT_REQUIRE(work.ptr != nullptr, "ras_setup: out of memory for the factorisation workspace");
    if (by_lines)
      factor_by_lines(R.get(), op->atab.as<double>(), d_lines.as<int32_t>(), d_line_lvl.as<int32_t>(), first, last,
                      work.as<double>(), d_status.as<int>(), s);
    else
      hipLaunchKernelGGL(factor_kernel, dim3(last - first), dim3(256), 0, s, op->d, R->d_subs.as<SubInfo>(),
                         R->d_shapes.as<ShapeInfo>(), R->d_lvl.as<int32_t>(), R->d_coords.as<uint64_t>(),
                         d_pstart.as<int16_t>(), d_pairs.as<uint8_t>(), first, work.as<double>(),
                         d_status.as<int>());
    STKKT_HIP(hipGetLastError());
    if (rp->precision == STKKT_F32) {
      hipLaunchKernelGGL(compact_kernel<float>, dim3(last - first, kCompactSplit), dim3(256), 0, s, R->d_subs.as<SubInfo>(),
                         R->d_shapes.as<ShapeInfo>(), R->d_lvl.as<int32_t>(), R->d_coords.as<uint64_t>(),
                         R->d_ctab.as<int32_t>(), first, work.as<double>(),
                         R->factors.as<float>());
    } else {
      hipLaunchKernelGGL(compact_kernel<double>, dim3(last - first, kCompactSplit), dim3(256), 0, s, R->d_subs.as<SubInfo>(),
                         R->d_shapes.as<ShapeInfo>(), R->d_lvl.as<int32_t>(), R->d_coords.as<uint64_t>(),
                         R->d_ctab.as<int32_t>(), first, work.as<double>(),
                         R->factors.as<double>());
    }
    STKKT_HIP(hipGetLastError());
    STKKT_HIP(hipStreamSynchronize(s));   // the workspace is released at the end of this scope
    first = last;
  }
  int status = 0;
  STKKT_HIP(hipMemcpy(&status, d_status.ptr, sizeof(int), hipMemcpyDeviceToHost));
  if (status != 0) throw Error(STKKT_EBREAKDOWN, "ras_setup: singular 3x3 pivot block in ILU(0)");
  return R.release();
}

void ras_export(const ras *R, int sub, double *out) {
  STKKT_REQUIRE(sub >= 0 && sub < R->nsub, "ras_export_factors: bad subdomain");
  STKKT_REQUIRE(!R->iluk, "ras_export_factors: ILU(k) factors have no 81-slot layout; use ras_export_factors_csr");
  const SubInfo &sd = R->subs[sub];
  const ShapeHost &sh = R->shapes[sd.shape];
  const int64_t nb = sh.felems;
  const bool f32 = R->params.precision == STKKT_F32;
  std::vector<double> buf((size_t)nb);
  if (f32) {
    std::vector<float> tmp((size_t)nb);
    STKKT_HIP(hipMemcpy(tmp.data(), R->factors.as<float>() + sd.fbase, sizeof(float) * tmp.size(),
                        hipMemcpyDeviceToHost));
    for (size_t i = 0; i < tmp.size(); ++i) buf[i] = tmp[i];
  } else {
    STKKT_HIP(hipMemcpy(buf.data(), R->factors.as<double>() + sd.fbase, sizeof(double) * buf.size(),
                        hipMemcpyDeviceToHost));
  }
  const int lx = sh.dims[0], ly = sh.dims[1], lz = sh.dims[2];
  const int32_t d32[4] = {sh.dims[0], sh.dims[1], sh.dims[2], sh.dims[3]};
  std::fill(out, out + (size_t)sh.vol * 729, 0.0);
  for (int L = 0; L < sh.nlev; ++L) {
    const int r0 = sh.lvl_start[L], R = sh.lvl_start[L + 1] - r0;
    for (int c = 0; c * 64 < R; ++c)
      for (int s = 0; s < 81; ++s) {
        int dx, dy, dz, dt;
        slot_off(s, dx, dy, dz, dt);
        const size_t i = (((size_t)L * sh.nchunk + c) * 81 + s) * 2;
        const int64_t off9 = sh.ctab[i], cnt = sh.ctab[i + 1];
        int64_t k = 0;
        for (int q = c * 64; q < std::min(R, c * 64 + 64); ++q) {
          int x, y, z, t;
          unpack(sh.coords[r0 + q], x, y, z, t);
          if (!inside(x + dx, y + dy, z + dz, t + dt, d32)) continue;
          const int64_t rho = x + (int64_t)lx * (y + (int64_t)ly * (z + (int64_t)lz * t));
          for (int e = 0; e < 9; ++e) out[rho * 729 + 9 * s + e] = buf[off9 + blk_pos(e, k, cnt)];
          ++k;
        }
        if (k != cnt) throw Error(STKKT_EINVAL, "ras_export_factors: inconsistent layout");
      }
  }
}

int64_t ras_sub_blocks(const ras *R, int sub) {
  STKKT_REQUIRE(sub >= 0 && sub < R->nsub, "ras_subdomain_blocks: bad subdomain");
  if (R->iluk) return iluk_subdomain_blocks(R, sub);
  return R->shapes[R->subs[sub].shape].nblocks;
}

void ras_export_csr(const ras *R, int sub, int32_t *indptr, int32_t *indices, double *blocks) {
  STKKT_REQUIRE(sub >= 0 && sub < R->nsub, "ras_export_factors_csr: bad subdomain");
  if (R->iluk) {
    iluk_export_csr(R, sub, indptr, indices, blocks);
    return;
  }
  const ShapeHost &sh = R->shapes[R->subs[sub].shape];
  std::vector<double> pad((size_t)sh.vol * 729);
  ras_export(R, sub, pad.data());
  const int lx = sh.dims[0], ly = sh.dims[1], lz = sh.dims[2];
  const int32_t d32[4] = {sh.dims[0], sh.dims[1], sh.dims[2], sh.dims[3]};
  int64_t k = 0;
  indptr[0] = 0;
  for (int rho = 0; rho < sh.vol; ++rho) {
    const int x = rho % lx, y = (rho / lx) % ly, z = (rho / (lx * ly)) % lz, t = rho / (lx * ly * lz);
    for (int s = 0; s < 81; ++s) {   // ascending slot = ascending column
      int dx, dy, dz, dt;
      slot_off(s, dx, dy, dz, dt);
      if (!inside(x + dx, y + dy, z + dz, t + dt, d32)) continue;
      indices[k] = (x + dx) + lx * ((y + dy) + ly * ((z + dz) + lz * (t + dt)));
      for (int e = 0; e < 9; ++e) blocks[9 * k + e] = pad[(size_t)rho * 729 + 9 * s + e];
      ++k;
    }
    indptr[rho + 1] = (int32_t)k;
  }
}

}  // namespace stkkt
