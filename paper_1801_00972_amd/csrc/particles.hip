// particles.hip -- particle kernels of the hot path (gfx950, wave64):
//   loading, the fused gather / leapfrog / wall / grain / collision / deposit
//   kernel in its FP64 and FP32R forms, the standalone deposit, and the
//   counting sort that keeps the particle arrays ordered by cell.
//
// Method (arXiv:1801.00972, Sec. III): CIC charge assignment and field gather
// on the cell corners, leapfrog Eq. (1)-(2), PPPM near-grain field Eq. (5)-(6)
// with dt_MD = dt/40, perfect absorption at electrodes and grains, binary
// collisions with the neutral reservoir (Table I) in null-collision form.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "device_common.hpp"
#include "launch.hpp"

namespace pic {

// constant memory: descriptors that no kernel writes, read by scalar loads
#define PIC_CONST __attribute__((address_space(4)))

// (the push packs them in nibbles: ST_ALIVE is 0)
enum { ST_ALIVE = 0, ST_WALL0 = 1, ST_WALL1 = 2, ST_GRAIN = 3, ST_NONE = 4, ST_BAD = 5, ST_MD = 6, ST_OUT = 7 };

// electrode test of a position already wrapped in x,y; a non-finite or
// out-of-range coordinate (which no valid input produces) removes the particle
template <typename H>
__device__ __forceinline__ int z_status(const double x[3], const H& S) {
  if (x[2] >= 0.0 && x[2] < (double)S.nz) {
    return (x[0] >= 0.0 && x[0] < (double)S.nx && x[1] >= 0.0 && x[1] < (double)S.ny) ? ST_ALIVE
                                                                                     : ST_BAD;
  }
  if (x[2] < 0.0) return ST_WALL0;
  if (x[2] >= (double)S.nz) return ST_WALL1;
  return ST_BAD;
}

constexpr int kBlock = 256;
constexpr int kPPT = 4;                   // consecutive particles per thread
constexpr int kChunk = kBlock * kPPT;     // slots one pass of a push block streams

// int32 cell index of the FP32R form: i | j << 10 | k << 20 (nx, ny <= 1024, nz < 2048);
// -1 marks an empty slot
__device__ __forceinline__ int cell_i(int c) { return c & 1023; }
__device__ __forceinline__ int cell_j(int c) { return (c >> 10) & 1023; }
__device__ __forceinline__ int cell_k(int c) { return c >> 20; }
__device__ __forceinline__ int pack_cell(int i, int j, int k) { return i | (j << 10) | (k << 20); }

// Blocks are dealt round-robin to the 8 XCDs; the items go to them in chunks of
// `chunk` consecutive ones, interleaved (XCD x takes chunks x, x + 8, ...): with
// a chunk of one z-layer of tiles every XCD works on layers spread over the whole
// height, so the particle density's variation along z (the sheaths) does not load
// some XCDs more than others, while neighbouring tiles of a layer share an L2.
// nb / 8 must be a multiple of chunk (then it is a permutation of [0, nb)).
__device__ __forceinline__ long xcd_interleave(long b, long chunk) {
  const long x = b % 8, i = b / 8;
  return ((i / chunk) * 8 + x) * chunk + i % chunk;
}

// ---------------------------------------------------------------- field loads
__device__ __forceinline__ void load_node(const double2* __restrict__ E, long n, double& ex,
                                          double& ey, double& ez) {
  const double2 a = E[2 * n], b = E[2 * n + 1];
  ex = a.x;
  ey = a.y;
  ez = b.x;
}
__device__ __forceinline__ void load_node(const float4* __restrict__ E, long n, double& ex,
                                          double& ey, double& ez) {
  const float4 a = E[n];
  ex = a.x;
  ey = a.y;
  ez = a.z;
}

// CIC gather in double precision at cell (i0,j0,k0), offsets (fx,fy,fz)
template <typename ET, typename H>
__device__ __forceinline__ void gather_d(const ET* __restrict__ E, const H& S, int i0,
                                         int j0, int k0, double fx, double fy, double fz,
                                         double out[3]) {
  const int i1 = i0 + 1 == S.nx ? 0 : i0 + 1;
  const int j1 = j0 + 1 == S.ny ? 0 : j0 + 1;
  const long r00 = (long)S.nx * j0 + (long)S.nxy * k0;
  const long r10 = (long)S.nx * j1 + (long)S.nxy * k0;
  const long r01 = r00 + S.nxy, r11 = r10 + S.nxy;
  const double wx[2] = {1.0 - fx, fx}, wy[2] = {1.0 - fy, fy}, wz[2] = {1.0 - fz, fz};
  const long base[4] = {r00, r10, r01, r11};
  out[0] = out[1] = out[2] = 0.0;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const double wyz = wy[t & 1] * wz[t >> 1];
    double ex, ey, ez;
    load_node(E, base[t] + i0, ex, ey, ez);
    out[0] += wx[0] * wyz * ex;
    out[1] += wx[0] * wyz * ey;
    out[2] += wx[0] * wyz * ez;
    load_node(E, base[t] + i1, ex, ey, ez);
    out[0] += wx[1] * wyz * ex;
    out[1] += wx[1] * wyz * ey;
    out[2] += wx[1] * wyz * ez;
  }
}

// ---------------------------------------------------------------- MD region
// index of cell (i, j, k) in the bounding box of the MD cubes, or -1
template <typename M>
__device__ __forceinline__ long md_box_index(const M& md, int nx, int ny, int i, int j,
                                             int k) {
  if (md.n_grains == 0) return -1;
  int a = i - md.bx0;
  if (a < 0) a += nx;
  if (a >= md.bsx) return -1;
  int b = j - md.by0;
  if (b < 0) b += ny;
  if (b >= md.bsy) return -1;
  const int c = k - md.bz0;
  if (c < 0 || c >= md.bsz) return -1;
  return ((long)c * md.bsy + b) * md.bsx + a;
}

template <typename M>
__device__ __forceinline__ uint32_t md_lookup(const M& md, int nx, int ny, int i, int j,
                                              int k) {
  const long bi = md_box_index(md, nx, ny, i, j, k);
  if (bi < 0) return 0u;
  const uint32_t cl = md.cell_list[bi];
  return (cl & 255u) ? cl : 0u;  // a cell of the box outside every cube has no grains
}

// 1 / sqrt(a), a > 0: the hardware estimate refined by two Newton steps
// y <- y (3 - a y^2) / 2 (each squares the relative error)
__device__ __forceinline__ double rsqrt_refined(double a) {
  double y = __builtin_amdgcn_rsq(a);
  y = y * (1.5 - 0.5 * a * y * y);
  y = y * (1.5 - 0.5 * a * y * y);
  return y;
}

__device__ __forceinline__ double wrap_coord(double X, int n) {
  if (X < 0.0) X += (double)n;
  else if (X >= (double)n) X -= (double)n;
  if (X >= (double)n) X -= (double)n;  // -tiny + n rounds to n
  if (X < 0.0 || X >= (double)n) X = X - (double)n * floor(X / (double)n);
  return X;
}

// The grain data that every sub-step reads, staged in LDS: positions in the frame
// of the MD box (x and y shifted by its origin, in [0, n)), and Q / (4 pi eps0
// dx^2).  raw: there are more grains than the stage holds; they are read from the
// tables, shifted and scaled where they are used.  The pointers are LDS pointers,
// not generic ones: a generic load waits for global memory too.
typedef const __attribute__((address_space(3))) double* LdsDoubles;
struct GrainView {
  LdsDoubles pos;  // [g][3]
  LdsDoubles Qc;   // [g]
  bool raw;
};

// the sum over the four lanes of a quad, in every lane (the two exchanges add
// the same pairs in each lane: equal bits)
__device__ __forceinline__ double quad_sum(double v) {
#define PIC_QUAD(ctrl)                                                                  \
  {                                                                                     \
    union {                                                                             \
      double d;                                                                         \
      int i[2];                                                                         \
    } a, b;                                                                             \
    a.d = v;                                                                            \
    b.i[0] = __builtin_amdgcn_mov_dpp(a.i[0], ctrl, 0xf, 0xf, true);                    \
    b.i[1] = __builtin_amdgcn_mov_dpp(a.i[1], ctrl, 0xf, 0xf, true);                    \
    v += b.d;                                                                           \
  }
  PIC_QUAD(0xB1)  // lanes 1 0 3 2
  PIC_QUAD(0x4E)  // lanes 2 3 0 1
#undef PIC_QUAD
  return v;
}
__device__ __forceinline__ int quad_min(int v) {
  v = min(v, __builtin_amdgcn_mov_dpp(v, 0xB1, 0xf, 0xf, true));
  return min(v, __builtin_amdgcn_mov_dpp(v, 0x4E, 0xf, 0xf, true));
}

// Sub-cycled PPPM motion near grains, Eq. (5)-(6): md_sub sub-steps of
// h = dt/md_sub with E = E_mesh - sum_g Q_g U_g + sum_g Q_g r / (4 pi eps0 r^3)
// over the grains whose cube holds the current cell; hit when |r| <= a (the
// first grain of the cell's list wins).  The first two terms are gathered from
// the cell's corrected node fields (built once per step by field_out_kernel),
// which are kept, with the cell's grains, until the cell changes.  x is in the
// MD box's frame (x and y minus its origin, in [0, n)): a cell's index in the
// box follows from the floor alone, and a separation inside the box needs no
// minimum image unless the box spans the period.
// kLanes = 4: the four lanes of a quad move one particle together, two corners
// of the cell and every fourth grain each; all its state is the same in each.  A
// sub-step is a serial chain, so a short list is bound by its length: 16x16x32
// cells, 5,500 particles, 62 to 72 us with one lane a particle, 35 us with four, 28 us
// with each lane's grains kept in registers and one test for the box's faces.  A
// long list (above kMdQuad particles) fills the chip with one lane each.
template <int kLanes, typename ET>
__device__ __forceinline__ int md_move(const ET* __restrict__ E, const MdTables& md,
                                       const GrainView& G, const SpeciesStep& S, double a2_cells,
                                       bool image, double x[3], double v[3], int& hit) {
  constexpr int kC = 8 / kLanes;            // corners of this lane
  constexpr int kG = kMdInline / kLanes;    // inline grains of this lane
  const int l = kLanes == 1 ? 0 : (int)threadIdx.x & (kLanes - 1);
  int ei = -1, ej = -1, ek = -1;
  double ec[kC][3];
  uint32_t cl = 0u;
  int cnt = 0;
  int gl[kG];
  // a quad's lanes keep their grains (box frame) and charges until the cell changes
  constexpr bool kKeep = kLanes == 4;
  double gk[kKeep ? kG : 1][4];
  double Ep[3];
  int first;  // list position of the first grain that holds the particle
  auto read_grain = [&](int g, double& g0, double& g1, double& g2, double& Qc) {
    if (G.raw) {
      g0 = md.gpos[3 * g] - md.bx0;
      g1 = md.gpos[3 * g + 1] - md.by0;
      g2 = md.gpos[3 * g + 2];
      if (g0 < 0.0) g0 += S.nx;
      if (g1 < 0.0) g1 += S.ny;
      Qc = md.Q[g] * S.coul_c;
    } else {
      g0 = G.pos[3 * g];
      g1 = G.pos[3 * g + 1];
      g2 = G.pos[3 * g + 2];
      Qc = G.Qc[g];
    }
  };
  auto pull = [&](int t, double g0, double g1, double g2, double Qc, bool test) {
    double r0 = x[0] - g0, r1 = x[1] - g1;
    const double r2 = x[2] - g2;
    if (image) {
      r0 = r0 > 0.5 * S.nx ? r0 - S.nx : (r0 < -0.5 * S.nx ? r0 + S.nx : r0);
      r1 = r1 > 0.5 * S.ny ? r1 - S.ny : (r1 < -0.5 * S.ny ? r1 + S.ny : r1);
    }
    const double rr = r0 * r0 + r1 * r1 + r2 * r2;
    if (test && rr <= a2_cells) first = min(first, t);
    if (Qc == 0.0) return;
    const double rs = rsqrt_refined(rr);
    const double inv = Qc * rs * rs * rs;
    Ep[0] += r0 * inv;
    Ep[1] += r1 * inv;
    Ep[2] += r2 * inv;
  };
  auto grain = [&](int t, int g, bool test) {
    double g0, g1, g2, Qc;
    read_grain(g, g0, g1, g2, Qc);
    pull(t, g0, g1, g2, Qc, test);
  };
  // position x_s, s = 0 .. md_sub: after a drift (s > 0) the hit test and,
  // before the next kick, the field, from one walk over the cell's grains
  for (int sub = 0;; ++sub) {
    const double f0 = floor(x[0]), f1 = floor(x[1]), f2 = floor(x[2]);
    const int i = (int)f0, j = (int)f1, k = (int)f2;
    if (i != ei || j != ej || k != ek) {
      ei = i;
      ej = j;
      ek = k;
      const int c = k - md.bz0;
      if ((unsigned)i < (unsigned)md.bsx && (unsigned)j < (unsigned)md.bsy &&
          (unsigned)c < (unsigned)md.bsz) {
        // (independent loads: one memory round trip)
        const long bi = ((long)c * md.bsy + j) * md.bsx + i;
        cl = md.cell_list[bi];
        const double* src = md.ecorr + bi * 24 + 3 * kC * l;
#pragma unroll
        for (int t = 0; t < kC; ++t) {
          ec[t][0] = src[3 * t];
          ec[t][1] = src[3 * t + 1];
          ec[t][2] = src[3 * t + 2];
        }
#pragma unroll
        for (int u = 0; u < kG; ++u) gl[u] = md.cell_first[bi * kMdInline + l + kLanes * u];
        cnt = (int)(cl & 255u);
        if constexpr (kKeep) {
#pragma unroll
          for (int u = 0; u < kG; ++u)
            if (l + kLanes * u < cnt) read_grain(gl[u], gk[u][0], gk[u][1], gk[u][2], gk[u][3]);
        }
      } else {
        cnt = 0;
        int i0 = i + md.bx0, j0 = j + md.by0;
        if (i0 >= S.nx) i0 -= S.nx;
        if (j0 >= S.ny) j0 -= S.ny;
        const int i1 = i0 + 1 == S.nx ? 0 : i0 + 1, j1 = j0 + 1 == S.ny ? 0 : j0 + 1;
#pragma unroll
        for (int t = 0; t < kC; ++t) {
          const int tt = kC * l + t;
          load_node(E, ((tt & 1) ? i1 : i0) + (long)S.nx * (((tt >> 1) & 1) ? j1 : j0) +
                           (long)S.nxy * (k + (tt >> 2)),
                    ec[t][0], ec[t][1], ec[t][2]);
        }
#pragma unroll
        for (int u = 0; u < kG; ++u) gl[u] = 0;
      }
    }
    const double fx = x[0] - f0, fy = x[1] - f1, fz = x[2] - f2;
    Ep[0] = Ep[1] = Ep[2] = 0.0;
    if constexpr (kLanes == 1) {
      const double wx[2] = {1.0 - fx, fx}, wy[2] = {1.0 - fy, fy}, wz[2] = {1.0 - fz, fz};
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const double w = wx[t & 1] * wy[(t >> 1) & 1] * wz[t >> 2];
        Ep[0] += w * ec[t][0];
        Ep[1] += w * ec[t][1];
        Ep[2] += w * ec[t][2];
      }
    } else {
      const double wyz = ((l & 1) ? fy : 1.0 - fy) * ((l & 2) ? fz : 1.0 - fz);
      const double w0 = (1.0 - fx) * wyz, w1 = fx * wyz;
#pragma unroll
      for (int a = 0; a < 3; ++a) Ep[a] = w0 * ec[0][a] + w1 * ec[1][a];
    }
    first = 256;
#pragma unroll
    for (int u = 0; u < kG; ++u) {
      if (l + kLanes * u >= cnt) continue;
      if constexpr (kKeep) pull(l + kLanes * u, gk[u][0], gk[u][1], gk[u][2], gk[u][3], sub > 0);
      else grain(l + kLanes * u, gl[u], sub > 0);
    }
    if (cnt > kMdInline)
      for (int t = kMdInline + l; t < cnt; t += kLanes) grain(t, md.grain_idx[(cl >> 8) + t], sub > 0);
    if constexpr (kLanes > 1) first = quad_min(first);
    if (first < 256) {
      hit = md.grain_idx[(cl >> 8) + first];
      return ST_GRAIN;
    }
    if (sub == S.md_sub) break;
    if constexpr (kLanes > 1) {
#pragma unroll
      for (int a = 0; a < 3; ++a) Ep[a] = quad_sum(Ep[a]);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      v[a] += S.qm_h * Ep[a];
      x[a] += v[a] * S.h_dx;
    }
    // (one test for the usual case, inside the box)
    if (!(x[0] >= 0.0 && x[0] < (double)S.nx && x[1] >= 0.0 && x[1] < (double)S.ny && x[2] > 0.0 &&
          x[2] < (double)S.nz)) {
      x[0] = wrap_coord(x[0], S.nx);
      x[1] = wrap_coord(x[1], S.ny);
      const int zs = z_status(x, S);
      if (zs != ST_ALIVE) return zs;
    }
  }
  return ST_ALIVE;
}

// The corrected node field of Eq. (5) at corner (ta, tb, tc) of MD box cell
// bi, whose lowest node is (i0, j0, k0): E_k(node) - sum_g Q_g U_g(node) over
// the cell's grains (cl: its list entry), in list order; E holds E_k(node).
__device__ __forceinline__ void md_corner(const MdTables& md, int nx, int ny, uint32_t cl, int i0,
                                          int j0, int k0, int ta, int tb, int tc, double E[3]) {
  const int cnt = (int)(cl & 255u);
  const int side = md.side;
  const long cube = (long)side * side * side;
  for (int u = 0; u < cnt; ++u) {
    const int g = md.grain_idx[(cl >> 8) + u];
    const double Q = md.Q[g];
    if (Q == 0.0) continue;
    int lx = i0 - (md.gcell[3 * g + 0] - md.cutoff);
    lx = ((lx % nx) + nx) % nx;
    int ly = j0 - (md.gcell[3 * g + 1] - md.cutoff);
    ly = ((ly % ny) + ny) % ny;
    const int lz = k0 - (md.gcell[3 * g + 2] - md.cutoff);
    const long l = ((long)(lz + tc) * side + (ly + tb)) * side + (lx + ta);
    const double* U = md.U + (long)g * 3 * cube;
    E[0] -= Q * U[l];
    E[1] -= Q * U[cube + l];
    E[2] -= Q * U[2 * cube + l];
  }
}

// The fields of a step in one launch.  Blocks [0, nbm): one thread per (MD box
// cell, corner) forms the corrected node field; E at the node is
// formed from psi and rounded to the storage type first, so it is what a read
// of E returns (these blocks come first: their dependent table loads then
// overlap the node blocks' streaming).  Blocks from nbm on: a thread takes one
// column of nodes through `planes` planes and writes phi (psi, the solve's interior
// potential, and the electrodes' lift) and E = -grad phi in the storage type, and
// clears the next step's charge accumulator (and the counts of its MD lists).
// With b (FP32R) the block's sums of (b - A psi)^2 and b^2 over its interior nodes
// go to partials: the six neighbours are at hand, so the residual costs one more
// read per node and no pass of its own.  Along the column the neighbours above
// and below and the lift's division are kept, and a large mesh leaves an eighth of
// the partial sums for the next solve to add up: 128x128x512 cells 167 -> 148 us here
// and 92 -> 42 in the solve, 64x64x256 18.5 -> 14.8 us; below 4,096 blocks of one
// plane each the chip has no work to spare, and a block takes one.
template <typename ET>
__global__ __launch_bounds__(256) void field_out_kernel(const double* __restrict__ psi,
                                                        double* __restrict__ phi,
                                                        ET* __restrict__ E,
                                                        unsigned long long* __restrict__ zero_next,
                                                        const double* __restrict__ b,
                                                        double* __restrict__ partials,
                                                        MdTables md, int* n_md0, int* n_md1,
                                                        int nx, int ny, int nz, double dx,
                                                        RfDrive rf, int nbm, int planes) {
  const double V = rf_voltage(rf);
  if (blockIdx.x == 0 && threadIdx.x == 0) *rf.next = *rf.step + 1u;
  if ((int)blockIdx.x >= nbm) {
    __shared__ double s_r[4], s_b[4];
    const int plane = nx * ny, per = (plane + 255) / 256;
    const int blk = (int)blockIdx.x - nbm, k0 = blk / per * planes;
    const int pn = (blk - blk / per * per) * 256 + (int)threadIdx.x;
    double rr = 0.0, bb = 0.0;
    if (pn < plane) {
      if (zero_next && k0 == 0 && pn == 0) {
        *n_md0 = 0;
        *n_md1 = 0;
      }
      const int y = pn / nx, x = pn - y * nx, row = y * nx;
      const int xp = row + (x + 1 == nx ? 0 : x + 1), xm = row + (x == 0 ? nx - 1 : x - 1);
      const int yp = (y + 1 == ny ? 0 : y + 1) * nx + x, ym = (y == 0 ? ny - 1 : y - 1) * nx + x;
      // psi at height h (interior: 1 .. nz - 1), the lift of its plane, and the lifted
      // potential: 0 and V on the electrodes
      auto psi_at = [&](int h, int i) { return h > 0 && h < nz ? psi[(long)(h - 1) * plane + i] : 0.0; };
      auto lift_of = [&](int h) { return V * (double)h / (double)nz; };
      auto lifted = [&](double q, double l, int h) { return h == 0 ? 0.0 : (h == nz ? V : q + l); };
      double l = lift_of(k0), qm = psi_at(k0 - 1, pn), q = psi_at(k0, pn);
      double cm = lifted(qm, lift_of(k0 - 1), k0 - 1), c = lifted(q, l, k0);
      const int k1 = min(k0 + planes, nz + 1);
      for (int k = k0; k < k1; ++k) {
        const long n = (long)k * plane + pn;
        const bool in = k > 0 && k < nz;
        const double qp = psi_at(k + 1, pn), ln = lift_of(k + 1), cp = lifted(qp, ln, k + 1);
        const double qxp = psi_at(k, xp), qxm = psi_at(k, xm), qyp = psi_at(k, yp), qym = psi_at(k, ym);
        if (zero_next) zero_next[n] = 0ull;
        phi[n] = c;
        const double ex = -(lifted(qxp, l, k) - lifted(qxm, l, k)) / (2.0 * dx);
        const double ey = -(lifted(qyp, l, k) - lifted(qym, l, k)) / (2.0 * dx);
        const double up = k == nz ? c : cp, dn = k == 0 ? c : cm;
        const double ez = -(up - dn) / (in ? 2.0 * dx : dx);
        if constexpr (std::is_same<ET, double2>::value) {
          E[2 * n] = make_double2(ex, ey);
          E[2 * n + 1] = make_double2(ez, 0.0);
        } else {
          E[n] = make_float4((float)ex, (float)ey, (float)ez, 0.0f);
        }
        if (b && in) {
          const double bi = b[n - plane];
          const double r = bi - (qxp + qxm + qyp + qym + qp + qm - 6.0 * q);
          rr += r * r;
          bb += bi * bi;
        }
        qm = q;
        q = qp;
        cm = c;
        c = cp;
        l = ln;
      }
    }
    if (!b) return;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      rr += __shfl_xor(rr, off, 64);
      bb += __shfl_xor(bb, off, 64);
    }
    if ((threadIdx.x & 63) == 0) {
      s_r[threadIdx.x >> 6] = rr;
      s_b[threadIdx.x >> 6] = bb;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      partials[2 * (long)blk] = s_r[0] + s_r[1] + s_r[2] + s_r[3];
      partials[2 * (long)blk + 1] = s_b[0] + s_b[1] + s_b[2] + s_b[3];
    }
    return;
  }
  const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long nbox = (long)md.bsx * md.bsy * md.bsz;
  if (gid >= 8 * nbox) return;
  const long bi = gid >> 3;
  const int t = (int)(gid & 7);
  const uint32_t cl = md.cell_list[bi];
  const int a = (int)(bi % md.bsx), bb = (int)((bi / md.bsx) % md.bsy);
  const int c = (int)(bi / ((long)md.bsx * md.bsy));
  const int i0 = (md.bx0 + a) % nx, j0 = (md.by0 + bb) % ny, k0 = md.bz0 + c;
  const int ta = t & 1, tb = (t >> 1) & 1, tc = t >> 2;
  const int in = i0 + ta == nx ? 0 : i0 + ta, jn = j0 + tb == ny ? 0 : j0 + tb;
  double En[3];
  node_field(psi, nx, ny, nz, dx, V, in, jn, k0 + tc, En[0], En[1], En[2]);
  if constexpr (!std::is_same<ET, double2>::value) {
#pragma unroll
    for (int q = 0; q < 3; ++q) En[q] = (double)(float)En[q];
  }
  md_corner(md, nx, ny, cl, i0, j0, k0, ta, tb, tc, En);
  double* dst = md.ecorr + bi * 24 + 3 * t;
  dst[0] = En[0];
  dst[1] = En[1];
  dst[2] = En[2];
}

// ---------------------------------------------------------------- collisions
// Null-collision MCC against the neutral reservoir: candidate iff Philox word 0
// is below the integer threshold of P' = 1 - exp(-n_g sigma g_cap dt); accept
// with probability g / g_cap.  e-Ar: elastic, isotropic in the CM frame with
// the neutral at rest.  Ar+-Ar: charge exchange, the ion takes the velocity of
// the neutral drawn from the 300 K reservoir.  T is the arithmetic of the
// form: double for FP64; float for FP32R, whose velocities are FP32 (its
// uniforms are the top 24 bits of the word plus one half, times 2^-24).
template <typename PT>
struct VelOf {
  using type = double;
};
template <>
struct VelOf<PartF32R> {
  using type = float;
};

template <typename T>
__device__ __forceinline__ T u01(uint32_t w) {
  if constexpr (sizeof(T) == 8) return u01_open(w);
  else return ((float)(w >> 8) + 0.5f) * 5.9604644775390625e-08f;
}

template <typename T>
__device__ __forceinline__ void normal_pair_t(uint32_t wa, uint32_t wb, T& n0, T& n1) {
  if constexpr (sizeof(T) == 8) {
    normal_pair(wa, wb, n0, n1);
  } else {
    const float r = sqrtf(-2.0f * logf(u01<float>(wa)));
    float sn, cs;
    sincosf(2.0f * (float)kPi * u01<float>(wb), &sn, &cs);
    n0 = r * cs;
    n1 = r * sn;
  }
}

// sigma of table column `col` at energy E (eV): linear between the grid
// points, the end values past them
template <typename H>
__device__ inline double xs_at(const H& S, int col, double E) {
  const double* x = S.xs;
  const double* t = S.xs + (long)col * S.xs_n;
  const int n = S.xs_n;
  if (E <= x[0]) return t[0];
  if (E >= x[n - 1]) return t[n - 1];
  int lo = 0, hi = n - 1;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (x[mid] <= E) lo = mid;
    else hi = mid;
  }
  const double f = (E - x[lo]) / (x[hi] - x[lo]);
  return t[lo] + f * (t[hi] - t[lo]);
}

// A candidate's collision with energy-dependent cross sections (FP64 in
// both forms): the process is picked by u1 against the cumulative
// g sigma_k(E) / (g sigma)_max, E the projectile's energy with the target at
// rest.  Electrons: elastic, then excitation (CM energy above E_ex; the CM
// energy drops by E_ex, isotropic scattering), then ionisation (CM energy
// above E_iz; what is left is shared, a uniform fraction s from
// Philox(id, k, IONIZE, 0) word 0 to the ejected electron, 1 - s to this one,
// which scatters isotropically; the event is recorded for ionize_kernel);
// ions: charge exchange, then isotropic elastic scattering in the CM frame of
// ion and neutral (equal masses).  Above the bound the collision happens
// (counted) and u1 splits the cross section.
template <typename T, typename H>
__device__ void collide_xs(const H& S, const uint4& r, const T vn[3], T v[3], bool& coll,
                           bool& capv, uint32_t id, long slot) {
  const double gx = (double)v[0] - (double)vn[0], gy = (double)v[1] - (double)vn[1],
               gz = (double)v[2] - (double)vn[2];
  const double g2 = gx * gx + gy * gy + gz * gz;
  const double g = sqrt(g2);
  const double E = 0.5 * g2 / fabs(S.qm);  // m g^2 / 2 in eV (|q| = e)
  double s1, s2, s3 = 0.0;
  if (S.sp == 0) {
    s1 = xs_at(S, 1, E);
    s2 = g2 > S.ex_g2 ? xs_at(S, 2, E) : 0.0;
    if (S.iz_ev && g2 > S.iz_g2) s3 = xs_at(S, 5, E);
  } else {
    s1 = xs_at(S, 3, E);
    s2 = xs_at(S, 4, E);
  }
  const double a1 = g * s1 / S.sg_max, a2 = g * (s1 + s2) / S.sg_max;
  const double a3 = g * (s1 + s2 + s3) / S.sg_max;
  const double u1 = u01_open(r.y);
  int proc;
  if (a3 > 1.0) {
    capv = true;
    const double x = u1 * (s1 + s2 + s3);
    proc = x < s1 ? 1 : (x < s1 + s2 ? 2 : 3);
  } else {
    proc = u1 < a1 ? 1 : (u1 < a2 ? 2 : (u1 < a3 ? 3 : 0));
  }
  if (proc == 0) return;
  coll = true;
  if (S.sp == 1 && proc == 1) {
    v[0] = vn[0];
    v[1] = vn[1];
    v[2] = vn[2];
    return;
  }
  const double cost = 1.0 - 2.0 * u01_open(r.z);
  const double sint = sqrt(fmax(0.0, 1.0 - cost * cost));
  double sp, cp;
  sincos(2.0 * kPi * u01_open(r.w), &sp, &cp);
  const double nh[3] = {sint * cp, sint * sp, cost};
  if (S.sp == 0) {
    double gp = proc == 2 ? sqrt(g2 - S.ex_g2) : g;
    if (proc == 3) {
      const double gsq = g2 - S.iz_g2;
      const uint4 w = philox4x32_10(id, *S.step, kIonize, 0u, S.key0, S.key1);
      gp = sqrt((1.0 - u01_open(w.x)) * gsq);
      const int e = atomicAdd(S.iz_cnt, 1);
      if (e < S.iz_cap) {
        IzEvent& ev = S.iz_ev[e];
        ev.id = id;
        ev.slot = (int32_t)slot;
        for (int a = 0; a < 3; ++a) ev.v[a] = (double)v[a];
        ev.gsq = gsq;
      }
    }
    for (int a = 0; a < 3; ++a) v[a] = (T)(S.mass_ratio_e * (double)v[a] + S.mass_ratio_n * gp * nh[a]);
  } else {
    for (int a = 0; a < 3; ++a) v[a] = (T)(0.5 * ((double)v[a] + (double)vn[a]) + 0.5 * g * nh[a]);
  }
}

template <typename T, typename H>
__device__ __forceinline__ void collide(const H& S, uint32_t id, T v[3], bool& coll,
                                        bool& capv, long slot) {
  if constexpr (sizeof(T) == 4) {
    // FP32R records: the collision in FP64 (2 % of the particles per step),
    // rounded once; a 24-bit uniform in the Box-Muller radius or the
    // scattering angle could put a tail draw 1e-4 off
    double vd[3] = {v[0], v[1], v[2]};
    collide<double>(S, id, vd, coll, capv, slot);
    if (coll) {
      v[0] = (T)vd[0];
      v[1] = (T)vd[1];
      v[2] = (T)vd[2];
    }
    return;
  }
  const uint4 r = philox4x32_10(id, *S.step, kColl, (uint32_t)S.sp, S.key0, S.key1);
  if ((uint64_t)r.x >= S.T_null) return;
  T vn[3] = {(T)0, (T)0, (T)0};
  if (S.sp == 1) {
    const uint4 q = philox4x32_10(id, *S.step, kNeutral, 1u, S.key0, S.key1);
    T n0, n1, n2, n3;
    normal_pair_t<T>(q.x, q.y, n0, n1);
    normal_pair_t<T>(q.z, q.w, n2, n3);
    const T vg = (T)S.vth_gas;
    vn[0] = vg * n0;
    vn[1] = vg * n1;
    vn[2] = vg * n2;
  }
  if (S.xs_n > 0) {
    collide_xs<T>(S, r, vn, v, coll, capv, id, slot);
    return;
  }
  const T gx = v[0] - vn[0], gy = v[1] - vn[1], gz = v[2] - vn[2];
  const T g = sqrt(gx * gx + gy * gy + gz * gz);
  const T ratio = g / (T)S.g_cap;
  bool accept;
  if (ratio > (T)1) {
    capv = true;
    accept = true;
  } else {
    accept = u01<T>(r.y) < ratio;
  }
  if (!accept) return;
  coll = true;
  if (S.sp == 0) {
    const T cost = (T)1 - (T)2 * u01<T>(r.z);
    const T sint = sqrt(fmax((T)0, (T)1 - cost * cost));
    T sp, cp;
    if constexpr (sizeof(T) == 8) sincos(2.0 * kPi * u01<T>(r.w), &sp, &cp);
    else sincosf(2.0f * (float)kPi * u01<T>(r.w), &sp, &cp);
    const T nh[3] = {sint * cp, sint * sp, cost};
    const T ae = (T)S.mass_ratio_e, an = (T)S.mass_ratio_n;
    for (int a = 0; a < 3; ++a) v[a] = ae * v[a] + an * g * nh[a];
  } else {
    v[0] = vn[0];
    v[1] = vn[1];
    v[2] = vn[2];
  }
}

// ---------------------------------------------------------------- deposit
// FP64 form: rho accumulates sign * W in units of the macro charge w e
// (cic_weights_d).
// FP32R form: the macro charge Qp (2^-32 e) split exactly into 8 non-negative
// parts, along x by q1 = (Q f24) >> 24 with f24 = floor(offset 2^24), then each
// half along y, each quarter along z; integer atomics, so the sum is exact and
// independent of order.
// (a b) >> 24 for 0 <= a < 2^39, 0 <= b < 2^24, exactly: a split at bit 24, so
// both products have 24-bit factors, which multiply at the full rate (a 32x32
// product takes four times as long)
__device__ __forceinline__ long long mul_shift24(long long a, uint32_t b) {
  const uint32_t lo = (uint32_t)a & 0xffffffu, hi = (uint32_t)(a >> 24) & 0xffffffu;
  const unsigned long long p = (unsigned long long)lo * b, q = (unsigned long long)hi * b;
  return (long long)(q + (uint32_t)(p >> 24));
}

__device__ __forceinline__ void split8(long long Q, float ox, float oy, float oz,
                                       long long part[8]) {
  // offsets in [0, 1): f24 in [0, 2^24), the parts stay in [0, Q]
  const uint32_t qx = (uint32_t)(ox * 16777216.0f) & 0xffffffu;
  const uint32_t qy = (uint32_t)(oy * 16777216.0f) & 0xffffffu;
  const uint32_t qz = (uint32_t)(oz * 16777216.0f) & 0xffffffu;
  long long ax[2];
  ax[1] = mul_shift24(Q, qx);
  ax[0] = Q - ax[1];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const long long y1 = mul_shift24(ax[a], qy);
    const long long yy[2] = {ax[a] - y1, y1};
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const long long z1 = mul_shift24(yy[b], qz);
      part[a + 2 * b] = yy[b] - z1;
      part[a + 2 * b + 4] = z1;
    }
  }
}

// ---------------------------------------------------------------- wave helpers
__device__ __forceinline__ int wave_sum(int v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
// ---------------------------------------------------------------- one particle
// FP32R: gather from the 8 node fields ec, kick Eq. (2), drift Eq. (1) in cell +
// offset form, periodic wrap; returns the electrode status
template <typename H>
__device__ __forceinline__ int push_one_f32(const H& S, const float ec[8][3], float o[3],
                                            float v[3], int& ci, int& cj, int& ck) {
  const float wx[2] = {1.0f - o[0], o[0]};
  const float wy[2] = {1.0f - o[1], o[1]};
  const float wz[2] = {1.0f - o[2], o[2]};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    float e = 0.0f;
#pragma unroll
    for (int t = 0; t < 8; ++t) e += wx[t & 1] * wy[(t >> 1) & 1] * wz[t >> 2] * ec[t][a];
    v[a] += S.qm_dt_f * e;
  }
  int d[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    float f = o[a] + v[a] * S.dt_dx_f;
    const float fl = floorf(f);
    f -= fl;
    d[a] = (int)fl;
    if (f >= 1.0f) {  // -tiny + 1 rounds to 1
      f = 0.0f;
      d[a] += 1;
    }
    o[a] = f;  // in [0, 1), or NaN
  }
  ci += d[0];
  cj += d[1];
  ck += d[2];
  // periodic wrap: one box length covers any move below it (the general
  // remainder only past that)
  if (ci < 0) ci += S.nx;
  else if (ci >= S.nx) ci -= S.nx;
  if (cj < 0) cj += S.ny;
  else if (cj >= S.ny) cj -= S.ny;
  if ((unsigned)ci >= (unsigned)S.nx || (unsigned)cj >= (unsigned)S.ny) {
    ci = ((ci % S.nx) + S.nx) % S.nx;
    cj = ((cj % S.ny) + S.ny) % S.ny;
  }
  return !(o[0] + o[1] + o[2] >= 0.0f) ? ST_BAD : (ck < 0 ? ST_WALL0 : (ck >= S.nz ? ST_WALL1 : ST_ALIVE));
}

// FP64: kick with the gathered field, drift, wrap; returns the electrode status
template <typename H>
__device__ __forceinline__ int push_one_f64(const H& S, const double Ep[3], double x[3],
                                            double v[3]) {
  v[0] += S.qm_dt * Ep[0];
  v[1] += S.qm_dt * Ep[1];
  v[2] += S.qm_dt * Ep[2];
  x[0] = wrap_coord(x[0] + v[0] * S.dt_dx, S.nx);
  x[1] = wrap_coord(x[1] + v[1] * S.dt_dx, S.ny);
  x[2] += v[2] * S.dt_dx;
  return z_status(x, S);
}

// ---------------------------------------------------------------- MD lists
// The dense MD list of the next step is formed at the end of this one.  The
// particles of a push block whose window meets the MD cubes' bounding box are
// looked through by the lists kernel (near_block, in slot order: the MD kernel
// is 1.5 times slower on a list in the order of arrival).  Elsewhere only a
// particle that has left its window can be in a cube: the kernel that moves it
// there (push, outliers, copy back, ionisation) appends it.  The re-binning,
// which moves the slots, lists its species anew.  A pass over the cells before
// each push instead was on the way to it and, as it had to look through every
// block that held a stray, read most slots (0.04 ms at 64x64x256, 32 ppc; 0.43
// ms at 128x128x512, 16 ppc).
template <typename M>
__device__ __forceinline__ bool in_md(const M& md, int nx, int ny, int c) {
  return md_lookup(md, nx, ny, cell_i(c), cell_j(c), cell_k(c)) != 0u;
}
__device__ __forceinline__ bool slot_alive(const PartF64& P, long p) { return P.z[p] >= 0.0; }
__device__ __forceinline__ bool slot_alive(const PartF32R& P, long p) { return P.cell[p] >= 0; }
__device__ __forceinline__ int slot_cell(const PartF64& P, long p) {
  return pack_cell((int)floor(P.x[p]), (int)floor(P.y[p]), (int)floor(P.z[p]));
}
__device__ __forceinline__ int slot_cell(const PartF32R& P, long p) { return P.cell[p]; }
// appends the value of each lane whose flag is set: one reservation for the wave
__device__ __forceinline__ void wave_append(bool flag, int32_t* list, int* count, int value) {
  const unsigned long long m = __ballot(flag);
  if (!m) return;
  const int lane = threadIdx.x & 63;
  const int leader = __ffsll((long long)m) - 1;
  int base = 0;
  if (lane == leader) base = atomicAdd(count, __popcll(m));
  base = __shfl(base, leader, 64);
  if (flag) list[base + __popcll(m & ((1ull << lane) - 1ull))] = value;
}

// ---------------------------------------------------------------- tile windows
// The arrays are binned by tiles of 4x4x4 cells.  One push block takes one
// tile: it stages the field on the tile's cells plus a margin of cells (the
// window) in LDS and accumulates its deposit there.  Particles that have
// drifted beyond the window since the last sort (fast electrons) are left to
// the outlier kernel, which gathers and deposits through global memory.
struct Tile {
  int x0, y0, k0;  // first node (x0, y0 may be negative: periodic)
  int tx, ty, tz;  // nodes per edge
  bool on;
  bool wraps;      // the window crosses the periodic seam in x or y
};

// the window of `span` tiles from (ti, tj, tk) (consecutive along x): their cells
// plus m cells on each side, in nodes; the margin shrinks until the window
// fits `cap` nodes
__host__ __device__ __forceinline__ Tile tile_window(int ti, int tj, int tk, int nx, int ny, int nz,
                                                     int margin, int cap, int span) {
  Tile w;
  w.on = false;
  w.wraps = false;
  w.x0 = w.y0 = w.k0 = 0;
  w.tx = w.ty = w.tz = 0;
  const int i0 = 4 * ti, ni = min(4 * span, nx - i0), j0 = 4 * tj, nj = min(4, ny - j0);
  const int k0 = 4 * tk, nk = min(4, nz - k0);
  for (int m = margin; m >= 0; --m) {
    int x0 = i0 - m, tx = ni + 2 * m + 1;
    if (ni + 2 * m >= nx) {
      x0 = 0;
      tx = nx + 1;
    }
    int y0 = j0 - m, ty = nj + 2 * m + 1;
    if (nj + 2 * m >= ny) {
      y0 = 0;
      ty = ny + 1;
    }
    const int klo = max(0, k0 - m), khi = min(nz - 1, k0 + nk - 1 + m);
    const int tz = khi - klo + 2;
    if (tx * ty * tz <= cap) {
      w.x0 = x0;
      w.y0 = y0;
      w.k0 = klo;
      w.tx = tx;
      w.ty = ty;
      w.tz = tz;
      w.on = true;
      w.wraps = x0 < 0 || x0 + tx - 1 >= nx || y0 < 0 || y0 + ty - 1 >= ny;
      return w;
    }
  }
  return w;
}

// the window of tiles t .. t + span - 1
template <typename WL>
__host__ __device__ __forceinline__ Tile make_tile(int t, const WL& L, int nx, int ny, int nz,
                                          int margin, int cap, int span = 1) {
  Tile w;
  w.on = false;
  w.wraps = false;
  w.x0 = w.y0 = w.k0 = 0;
  w.tx = w.ty = w.tz = 0;
  // a padding tile of the grid (its slots, if any, hold particles made by
  // ionisation since the last re-binning): no window, every particle takes
  // the global-memory paths
  if (t >= L.ntx * L.nty * L.ntz) return w;
  return tile_window(t % L.ntx, (t / L.ntx) % L.nty, t / (L.ntx * L.nty), nx, ny, nz, margin, cap, span);
}
// tile-local index of the cell's lower corner node, or -1 if the cell's 8
// nodes are not all in the tile
__device__ __forceinline__ int tile_cell(const Tile& t, int i, int j, int k, int nx, int ny) {
  if (!t.on) return -1;
  int lx = i - t.x0;
  int ly = j - t.y0;
  if (t.wraps) {  // (block-uniform)
    if (lx >= nx) lx -= nx;
    else if (lx < 0) lx += nx;
    if (ly >= ny) ly -= ny;
    else if (ly < 0) ly += ny;
  }
  const int lz = k - t.k0;
  // (unsigned: a negative index, possible without the wrap, is out too)
  if ((unsigned)lx > (unsigned)(t.tx - 2) || (unsigned)ly > (unsigned)(t.ty - 2) ||
      (unsigned)lz > (unsigned)(t.tz - 2))
    return -1;
  // (24-bit products: a 32-bit one takes four times as long)
  return (int)(__umul24(__umul24((unsigned)lz, (unsigned)t.ty) + (unsigned)ly, (unsigned)t.tx)) + lx;
}

// a / b for 0 <= a < 2^24 without an integer divide (rb = 1/b)
__device__ __forceinline__ int qdiv(int a, int b, float rb) {
  int q = (int)((float)a * rb);
  if (q * b > a) --q;
  else if ((q + 1) * b <= a) ++q;
  return q;
}

// global node of tile entry t
__device__ __forceinline__ long tile_node(const Tile& T, int t, float rtx, float rtxy, int nx,
                                          int ny, long nxy) {
  const int lz = qdiv(t, T.tx * T.ty, rtxy);
  const int r = t - lz * T.tx * T.ty;
  const int ly = qdiv(r, T.tx, rtx);
  const int lx = r - ly * T.tx;
  int gi = T.x0 + lx;
  if (gi < 0) gi += nx;
  else if (gi >= nx) gi -= nx;
  if (gi < 0 || gi >= nx) gi = ((gi % nx) + nx) % nx;
  int gj = T.y0 + ly;
  if (gj < 0) gj += ny;
  else if (gj >= ny) gj -= ny;
  if (gj < 0 || gj >= ny) gj = ((gj % ny) + ny) % ny;
  return gi + (long)nx * gj + nxy * (T.k0 + lz);
}

template <typename A>
__device__ __forceinline__ void atomic_add_acc(A* p, A v) {
  if constexpr (std::is_same<A, long long>::value)
    atomicAdd((unsigned long long*)p, (unsigned long long)v);
  else
    unsafeAtomicAdd(p, v);
}

// the 8 corner contributions of one cell into the tile (lbase >= 0) or to global
template <typename A, typename H>
__device__ __forceinline__ void corner_add(const Tile& T, int lbase, A* s_rho, A* __restrict__ rho,
                                           const H& S, int i, int j, int k,
                                           const A acc[8]) {
  if (lbase >= 0) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int off = (t & 1) + T.tx * (((t >> 1) & 1) + T.ty * (t >> 2));
      if constexpr (std::is_same<A, long long>::value)
        atomicAdd((unsigned long long*)&s_rho[lbase + off], (unsigned long long)acc[t]);
      else
        atomicAdd(&s_rho[lbase + off], acc[t]);
    }
  } else {
    const int i1 = i + 1 == S.nx ? 0 : i + 1;
    const int j1 = j + 1 == S.ny ? 0 : j + 1;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const long node = ((t & 1) ? i1 : i) + (long)S.nx * (((t >> 1) & 1) ? j1 : j) +
                        (long)S.nxy * (k + (t >> 2));
      atomic_add_acc(&rho[node], acc[t]);
    }
  }
}

// one particle's CIC charge straight to the global mesh (particles outside their tile's window)
template <typename H>
__device__ __forceinline__ void deposit_global_fixed(long long* __restrict__ rho, const H& S, int i, int j, int k,
                                                     float ox, float oy, float oz) {
  long long part[8];
  split8(S.Qp, ox, oy, oz, part);
#pragma unroll
  for (int t = 0; t < 8; ++t) part[t] *= S.isign;
  Tile none{};
  corner_add<long long>(none, -1, nullptr, rho, S, i, j, k, part);
}

__device__ __forceinline__ void cic_weights_d(double fx, double fy, double fz, double s,
                                              double w[8]) {
  const double wx[2] = {1.0 - fx, fx}, wy[2] = {1.0 - fy, fy}, wz[2] = {1.0 - fz, fz};
#pragma unroll
  for (int t = 0; t < 8; ++t) w[t] = s * wx[t & 1] * wy[(t >> 1) & 1] * wz[t >> 2];
}

// append to a list segment: one LDS atomic per wave
__device__ __forceinline__ void chunk_append(bool flag, int32_t* seg, int* s_n, int value) {
  const unsigned long long m = __ballot(flag);
  if (!m) return;
  const int lane = threadIdx.x & 63;
  const int leader = __ffsll((long long)m) - 1;
  int base = 0;
  if (lane == leader) base = atomicAdd(s_n, __popcll(m));
  base = __shfl(base, leader, 64);
  if (flag) seg[base + __popcll(m & ((1ull << lane) - 1ull))] = value;
}

// block-level tallies: wave sums into LDS; thread 0 then adds them to the
// tile's own accumulators (each tile has one writer per kernel: no atomics)
__device__ __forceinline__ void tally_add(unsigned* s_t, int which, int v) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0 && v) atomicAdd(&s_t[which], (unsigned)v);
}
__device__ __forceinline__ void tally_store(unsigned* s_t, unsigned long long* tally) {
  if (threadIdx.x != 0) return;
  s_t[TL_DEAD] = s_t[TL_W0] + s_t[TL_W1] + s_t[TL_BAD];
  for (int w = 0; w < TL_N; ++w)
    if (s_t[w]) tally[w] += s_t[w];
}

__device__ __forceinline__ PartF32R desc_records(const PIC_CONST PushDescF32* d) {
  return PartF32R{d->P.cell, d->P.ox, d->P.oy, d->P.oz, d->P.vx, d->P.vy, d->P.vz, d->P.id};
}
__device__ __forceinline__ PartF64 desc_records(const PIC_CONST PushDescF64* d) {
  return PartF64{d->P.x, d->P.y, d->P.z, d->P.vx, d->P.vy, d->P.vz, d->P.id};
}
// whether the packed cell lies in an MD cube, for the push's inner loop: the
// tables are read here, not kept in registers
template <typename Desc>
__device__ __forceinline__ bool push_in_md(const PIC_CONST Desc* d, int c) {
  return in_md(d->md, d->S.nx, d->S.ny, c);
}
// one run of same-cell charge parts (magnitudes) into the window, or, outside
// it, with the species' sign straight to the global mesh (*s_far is set if that
// cell lies in an MD cube)
__device__ __forceinline__ void deposit_run(const Tile& tile, long long* s_rho,
                                            const PIC_CONST PushDescF32* d, int nx, int ny, int c,
                                            long long acc[8], int* s_far) {
  const int lb = tile_cell(tile, cell_i(c), cell_j(c), cell_k(c), nx, ny);
  if (lb >= 0) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int off = (t & 1) + tile.tx * (((t >> 1) & 1) + tile.ty * (t >> 2));
      atomicAdd((unsigned long long*)&s_rho[lb + off], (unsigned long long)acc[t]);
    }
    return;
  }
  if (push_in_md(d, c)) *s_far = 1;
  if (d->S.isign < 0) {
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] = -acc[t];
  }
  corner_add<long long>(tile, -1, s_rho, d->rho, d->S, cell_i(c), cell_j(c), cell_k(c), acc);
}
// A push block away from the MD cubes moved a particle into one (rare): its
// slots [beg, end) are looked through again, and those in a cube that did not
// start there (as ~slot in the out list's n_out entries) listed for the next step.
template <typename PT, typename WL, typename M>
__device__ void list_far(const PT& P, const WL& L, const M& md, int nx, int ny, int beg,
                         int end, int n_out) {
  for (int p = beg + (int)threadIdx.x; p < end; p += kBlock) {
    if (!slot_alive(P, p) || !in_md(md, nx, ny, slot_cell(P, p))) continue;
    bool started = false;
    for (int t = 0; t < n_out && !started; ++t) started = L.out[beg + t] == ~p;
    if (!started) L.md_next[atomicAdd(L.n_md_next, 1)] = p;
  }
}

// The events of a push pass that few particles have, out of the inner loop's
// way: st packs the status of a lane's kPPT slots (from p0) in nibbles.  Counts
// the absorbed and the bad ones, the MD particles and those outside the window,
// lists the latter two where they are to be listed, and marks both in the mask
// of a block near the MD cubes.  The whole wave calls it.
template <typename WL>
__device__ __forceinline__ void push_events(unsigned st, int p0, bool have, bool md_near,
                                            const WL& L, int32_t* out, int* s_nout,
                                            unsigned* s_tally) {
  unsigned mask = 0;
#pragma unroll
  for (int q = 0; q < kPPT; ++q) {
    const int e = (int)((st >> (4 * q)) & 15u);
    if (!__any(e != ST_ALIVE && e != ST_NONE)) continue;
    const bool md = e == ST_MD, o = e == ST_OUT;
    const unsigned long long w0 = __ballot(e == ST_WALL0), w1 = __ballot(e == ST_WALL1),
                             bad = __ballot(e == ST_BAD), m = __ballot(md), f = __ballot(o);
    if ((threadIdx.x & 63) == 0) {
      if (w0) atomicAdd(&s_tally[TL_W0], (unsigned)__popcll(w0));
      if (w1) atomicAdd(&s_tally[TL_W1], (unsigned)__popcll(w1));
      if (bad) atomicAdd(&s_tally[TL_BAD], (unsigned)__popcll(bad));
      if (m) atomicAdd(&s_tally[TL_MD], (unsigned)__popcll(m));
      if (f) atomicAdd(&s_tally[TL_FALL], (unsigned)__popcll(f));
    }
    const bool far_md = md && !md_near;
    chunk_append(o || far_md, out, s_nout, far_md ? ~(p0 + q) : p0 + q);
    mask |= (md ? 1u << q : 0u) | (o ? 16u << q : 0u);
  }
  if (md_near && have && mask) L.mask[p0 / kPPT] = (uint8_t)mask;
}

// whether any cell of the window lies in the bounding box of the MD cubes
// (periodic in x, y)
template <typename M>
__host__ __device__ __forceinline__ bool window_meets_md(const Tile& w, const M& md, int nx, int ny) {
  if (md.n_grains == 0) return false;
  if (!w.on) return true;
  const int wx = w.tx - 1, wy = w.ty - 1;  // cells of the window per axis
  int dx = (w.x0 - md.bx0) % nx;
  if (dx < 0) dx += nx;
  int dy = (w.y0 - md.by0) % ny;
  if (dy < 0) dy += ny;
  const bool mx = wx >= nx || dx < md.bsx || dx + wx > nx;
  const bool my = wy >= ny || dy < md.bsy || dy + wy > ny;
  const bool mz = w.k0 < md.bz0 + md.bsz && md.bz0 < w.k0 + w.tz - 1;
  return mx && my && mz;
}

// ---------------------------------------------------------------- push, FP32R
// One block streams the slots of its tile, 1024 per pass, four consecutive
// slots per thread with 16-byte loads and stores, and updates them in place:
// gather from the LDS field window (the 8 node fields are reused while
// consecutive particles share a cell), kick Eq. (2), drift Eq. (1) in cell +
// offset form, periodic wrap, electrode absorption, collision candidate test;
// the new positions are deposited into the LDS window (per-thread sums over a
// run of particles in one cell first), whose occupied nodes are then added to
// rho.  Particles starting inside an MD cube are left untouched (their list
// is there when the step starts, and the sub-cycled kernel moves them meanwhile
// into the other record buffer); the block collides its candidates at its end (cand_collide).
constexpr int kWinF32 = 1331;  // window capacity (nodes): a tile with a 3-cell margin

// The FP32R push streams the particle records once per step in each direction
// and they are not reread before they would have left the caches: their
// 16-byte loads and stores carry the non-temporal hint, which keeps the field
// and deposit windows and the lists cached instead.  (Measured: faster here;
// slower for the FP64 records' 16-byte pairs and the re-binning's 4-byte
// scatter, which keep the default.)
// the kPPT consecutive values of one field at group g (FP32R push records)
typedef int viP __attribute__((ext_vector_type(kPPT)));
typedef float vfP __attribute__((ext_vector_type(kPPT)));
typedef unsigned vuP __attribute__((ext_vector_type(kPPT)));
template <typename V, typename T>
__device__ __forceinline__ V nt_loadP(const T* p, long g) {
  return __builtin_nontemporal_load(reinterpret_cast<const V*>(p) + g);
}
template <typename V, typename T>
__device__ __forceinline__ void nt_store4(T* p, long g4, V v) {
  __builtin_nontemporal_store(v, reinterpret_cast<V*>(p) + g4);
}

// The collision candidates of a push block, kept in LDS with what the collision
// needs: the block collides them after its last pass, 64 to a wave, and writes
// the velocities back.  A kernel of its own after the push gathered id and
// velocity of every candidate (2 % of the electrons) from memory again, half of
// all the cache lines of those arrays: 64x64x256 75 us, 128x128x512 0.9 ms a
// step.  Candidates beyond the stage go to the list in memory.
template <typename V, int N>
struct CandStage {
  V v[3][N];
  uint32_t id[N];
  int slot[N];
};
constexpr int kCandF32 = 368;  // (39.4 KB of LDS in all: four blocks a CU)
constexpr int kCandF64 = 320;  // (52.4 KB: three)

// the candidates of a wave's slots p0 .. p0 + kPPT - 1 (bit q of cm) into the
// stage or, past it, the list: one reservation.  The whole wave calls it.
template <typename V, int N>
__device__ __forceinline__ void cand_append(unsigned cm, CandStage<V, N>& cs, int32_t* list, int* s_n,
                                            int p0, const uint32_t id[kPPT], const V v[kPPT][3]) {
  unsigned long long m[kPPT];
  int total = 0;
#pragma unroll
  for (int q = 0; q < kPPT; ++q) {
    m[q] = __ballot((cm >> q) & 1u);
    total += __popcll(m[q]);
  }
  const int lane = threadIdx.x & 63;
  int base = 0;
  if (lane == 0) base = atomicAdd(s_n, total);
  base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
  for (int q = 0; q < kPPT; ++q) {
    if ((cm >> q) & 1u) {
      const int at = base + __popcll(m[q] & ((1ull << lane) - 1ull));
      if (at < N) {
        cs.v[0][at] = v[q][0];
        cs.v[1][at] = v[q][1];
        cs.v[2][at] = v[q][2];
        cs.id[at] = id[q];
        cs.slot[at] = p0 + q;
      } else {
        list[at - N] = p0 + q;
      }
    }
    base += __popcll(m[q]);
  }
}
// collides the staged candidates (after a barrier) and writes those that did
// collide back to P
template <typename PT, typename H, typename V, int N>
__device__ __forceinline__ void cand_collide(const PT& P, const H& S, const CandStage<V, N>& cs,
                                             int n, unsigned* s_tally) {
  n = min(n, N);
  if (((int)threadIdx.x & ~63) >= n) return;  // (wave-uniform)
  int n_coll = 0, n_cap = 0;
  for (int i = (int)threadIdx.x; i < n; i += kBlock) {
    bool coll = false, capv = false;
    V v[3] = {cs.v[0][i], cs.v[1][i], cs.v[2][i]};
    const int p = cs.slot[i];
    collide(S, cs.id[i], v, coll, capv, (long)p);
    if (coll) {
      P.vx[p] = v[0];
      P.vy[p] = v[1];
      P.vz[p] = v[2];
    }
    n_coll += coll;
    n_cap += capv;
  }
  tally_add(s_tally, TL_COLL, n_coll);
  tally_add(s_tally, TL_CAP, n_cap);
}

// LDS of one push block (FP32R)
template <typename PT, bool kMove>
struct PushSmem;
template <bool kMove>
struct PushSmem<PartF32R, kMove> {
  float4 E[kWinF32];
  long long rho[kWinF32];
  unsigned tally[TL_N];
  int ncoll, nout, far;
  CandStage<float, kCandF32> cand;
};

// A block takes `span` tiles that are consecutive along x (1 or 2): their
// slots are one contiguous range and they share one window; the lists of the
// span go to the first tile's segments, the others' counts are zero.
struct PushHot {  // what the inner loop needs of a SpeciesStep
  int nx, ny, nz;
  float qm_dt_f, dt_dx_f;
};
template <bool kMove>
__device__ __forceinline__ void push_tile(const PIC_CONST PushDescF32* d, int tidx, int span,
                                          PushSmem<PartF32R, kMove>& sm) {
  const int beg = d->L.tstart[tidx], end = d->L.tstart[tidx + span];
  if (kMove && threadIdx.x < span) {
    d->L.coll_cnt[tidx + threadIdx.x] = 0;
    d->L.out_cnt[tidx + threadIdx.x] = 0;
  }
  if (beg >= end) return;
  const PushHot S{d->S.nx, d->S.ny, d->S.nz, d->S.qm_dt_f, d->S.dt_dx_f};
  const Tile tile = make_tile(tidx, d->L, S.nx, S.ny, S.nz, d->S.margin, kWinF32, span);
  const int vol = tile.on ? tile.tx * tile.ty * tile.tz : 0;
  const float rtx = 1.0f / (float)max(tile.tx, 1), rtxy = 1.0f / (float)max(tile.tx * tile.ty, 1);
  for (int t = threadIdx.x; t < vol; t += kBlock) {
    if (kMove) sm.E[t] = d->E[tile_node(tile, t, rtx, rtxy, S.nx, S.ny, d->S.nxy)];
    sm.rho[t] = 0;
  }
  if (threadIdx.x < TL_N) sm.tally[threadIdx.x] = 0;
  if (threadIdx.x == 0) {
    sm.ncoll = 0;
    sm.nout = 0;
    sm.far = 0;
  }
  // MD cubes near the window: only then does every particle need the lookup
  const bool md_near = window_meets_md(tile, d->md, S.nx, S.ny);
  const PartF32R P = desc_records(d);
  int32_t* const coll = d->L.coll + beg;
  int32_t* const out = d->L.out + beg;
  const float vfast2 = d->S.vfast2_f;
  const uint32_t step = kMove ? *d->S.step : 0u, key0 = d->S.key0, key1 = d->S.key1, sp = (uint32_t)d->S.sp;
  // a candidate has word 0 < T_null (at most 2^32), that is <= T_null - 1
  const bool cand_on = d->S.T_null != 0;
  const uint32_t T_last = (uint32_t)(d->S.T_null - 1);
  const long long Qp = d->S.Qp;
  __syncthreads();
  int n_fast = 0;
  for (int base = beg; base < end; base += kChunk) {
    // tile ranges are multiples of 4 slots: a thread's kPPT slots are all in
    // the tile or all beyond it
    const int p0 = base + kPPT * (int)threadIdx.x;
    const bool have = p0 < end;
    const long g4 = p0 / kPPT;
    int cell[kPPT];
    float o[kPPT][3], v[kPPT][3];
    uint32_t id[kPPT];
    {
      viP c4 = -1;
      vfP X4 = 0.0f, Y4 = 0.0f, Z4 = 0.0f, U4 = 0.0f, V4 = 0.0f, W4 = 0.0f;
      vuP I4 = 0u;
      if (have) {
        c4 = nt_loadP<viP>(P.cell, g4);
        X4 = nt_loadP<vfP>(P.ox, g4);
        Y4 = nt_loadP<vfP>(P.oy, g4);
        Z4 = nt_loadP<vfP>(P.oz, g4);
        U4 = nt_loadP<vfP>(P.vx, g4);
        V4 = nt_loadP<vfP>(P.vy, g4);
        W4 = nt_loadP<vfP>(P.vz, g4);
        I4 = nt_loadP<vuP>(P.id, g4);
      }
#pragma unroll
      for (int q = 0; q < kPPT; ++q) {
        cell[q] = c4[q];
        o[q][0] = X4[q];
        o[q][1] = Y4[q];
        o[q][2] = Z4[q];
        v[q][0] = U4[q];
        v[q][1] = V4[q];
        v[q][2] = W4[q];
        id[q] = I4[q];
      }
    }
    // the statuses, in nibbles; live: bit q set for a particle that moved and is
    // alive (its charge is deposited)
    unsigned st = 0, live = 0;
#pragma unroll
    for (int q = 0; q < kPPT; ++q) {
      if (!kMove) {
        if (cell[q] >= 0) live |= 1u << q;
        continue;
      }
      int ci = cell_i(cell[q]), cj = cell_j(cell[q]), ck = cell_k(cell[q]);
      const int lb = tile_cell(tile, ci, cj, ck, S.nx, S.ny);
      int e = cell[q] < 0 ? ST_NONE : (lb < 0 ? ST_OUT : ST_ALIVE);
      // outside the window: left for the outlier kernel (no global gather here,
      // so no wave waits on a dependent memory round trip); in an MD cube: left
      // for the sub-cycled one
      if (cell[q] >= 0 && (md_near || lb < 0) && push_in_md(d, cell[q])) e = ST_MD;
      if (e == ST_ALIVE) {
        float ec[8][3];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const float4 f = sm.E[lb + (t & 1) + tile.tx * (((t >> 1) & 1) + tile.ty * (t >> 2))];
          ec[t][0] = f.x;
          ec[t][1] = f.y;
          ec[t][2] = f.z;
        }
        e = push_one_f32(S, ec, o[q], v[q], ci, cj, ck);
        cell[q] = e == ST_ALIVE ? pack_cell(ci, cj, ck) : -1;
        n_fast += v[q][0] * v[q][0] + v[q][1] * v[q][1] + v[q][2] * v[q][2] >= vfast2;
        live |= (e == ST_ALIVE ? 1u : 0u) << q;
      }
      st |= (unsigned)e << (4 * q);
    }
    if (kMove) {
      // collision candidates of the survivors: word 0 of Philox(id, k, COLL, s).
      // (the key passes through the opaque asm so that its 20 round keys are
      // formed per pass, not held in scalar registers across the loop)
      if (cand_on) {
        uint32_t w0[kPPT], k0 = key0, k1 = key1;
        asm volatile("" : "+s"(k0), "+s"(k1));
        philox_word0<kPPT>(id, step, kColl, sp, k0, k1, w0);
        unsigned cm = 0;
#pragma unroll
        for (int q = 0; q < kPPT; ++q) cm |= (w0[q] <= T_last ? 1u : 0u) << q;
        cm &= live;
        if (__any(cm)) cand_append(cm, sm.cand, coll, &sm.ncoll, p0, id, v);
      }
      if (md_near && have) d->L.mask[g4] = 0;
      if (__any((st & 0xbbbbu) != 0u))  // neither alive nor an empty slot
        push_events(st, p0, have, md_near, d->L, out, &sm.nout, sm.tally);
      if (have) {
        viP c;
        vfP a0, a1, a2, b0, b1, b2;
#pragma unroll
        for (int q = 0; q < kPPT; ++q) {
          c[q] = cell[q];
          a0[q] = o[q][0];
          a1[q] = o[q][1];
          a2[q] = o[q][2];
          b0[q] = v[q][0];
          b1[q] = v[q][1];
          b2[q] = v[q][2];
        }
        nt_store4<viP>(P.cell, g4, c);
        nt_store4<vfP>(P.ox, g4, a0);
        nt_store4<vfP>(P.oy, g4, a1);
        nt_store4<vfP>(P.oz, g4, a2);
        nt_store4<vfP>(P.vx, g4, b0);
        nt_store4<vfP>(P.vy, g4, b1);
        nt_store4<vfP>(P.vz, g4, b2);
      }
    }

    // deposit of rho_{k+1}
    long long acc[8];
    int acc_cell = -1;
#pragma unroll
    for (int q = 0; q < kPPT; ++q) {
      if (!((live >> q) & 1u)) continue;
      long long part[8];
      split8(Qp, o[q][0], o[q][1], o[q][2], part);
      if (cell[q] == acc_cell) {
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[t] += part[t];
      } else {
        if (acc_cell >= 0) deposit_run(tile, sm.rho, d, S.nx, S.ny, acc_cell, acc, &sm.far);
        acc_cell = cell[q];
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[t] = part[t];
      }
    }
    if (acc_cell >= 0) deposit_run(tile, sm.rho, d, S.nx, S.ny, acc_cell, acc, &sm.far);
  }
  if (kMove) tally_add(sm.tally, TL_FAST, n_fast);
  __syncthreads();
  if (kMove) cand_collide(P, d->S, sm.cand, sm.ncoll, sm.tally);
  // the window holds the magnitudes; the species' sign is applied here
  const int isign = (int)d->S.isign;
  const long nxy = d->S.nxy;
  long long* const rho = d->rho;
  const float qtx = 1.0f / (float)max(tile.tx, 1), qtxy = 1.0f / (float)max(tile.tx * tile.ty, 1);
  for (int t = threadIdx.x; t < vol; t += kBlock) {
    const long long val = sm.rho[t];
    if (val != 0)
      atomicAdd((unsigned long long*)&rho[tile_node(tile, t, qtx, qtxy, S.nx, S.ny, nxy)],
                (unsigned long long)(isign < 0 ? -val : val));
  }
  if (kMove) {
    if (threadIdx.x == 0) {
      d->L.coll_cnt[tidx] = max(0, sm.ncoll - kCandF32);
      d->L.out_cnt[tidx] = sm.nout;
    }
    __syncthreads();
    tally_store(sm.tally, d->L.tally + (long)TL_N * tidx);
    if (sm.far && !md_near) list_far(P, d->L, d->md, S.nx, S.ny, beg, end, sm.nout);
  }
}

// Both species in one launch (blocks [0, nb) electrons): they meet only in the
// atomically summed charge, one launch has one tail, and on a small box a second
// stream's fork and join cost as much as the push itself (8 us each).
// (at most 128 VGPRs: four waves per SIMD, which the streaming needs)
template <bool kMove>
__global__ __launch_bounds__(kBlock, 4) void push_f32r_kernel(const PushDescF32* descs, int nb,
                                                           int span, int chunk) {
  __shared__ PushSmem<PartF32R, kMove> sm;
  const int sp = (int)blockIdx.x >= nb ? 1 : 0, b = (int)blockIdx.x - sp * nb;
  push_tile<kMove>((const PIC_CONST PushDescF32*)(descs + sp), span * (int)xcd_interleave(b, chunk), span, sm);
}

// ---------------------------------------------------------------- push, ensemble
// One launch over the tile spans of every (replica, species) of an ensemble:
// block i takes work item i, of descriptor lo with start[lo] <= i < start[lo + 1]
// (each descriptor has a multiple of 8 items, so item i runs on XCD i mod 8 as
// the tile interleave expects).  A block an item, dealt by the hardware as
// blocks end: a persistent grid drawing items from queues kept its loop's state
// through every tile (30 spilled registers) and took 2.77 ms a step where this
// takes 2.32 ms (six replicas of 1.5e8 particles in all).
__global__ __launch_bounds__(kBlock, 4) void push_batch_f32r_kernel(const PushDescF32* descs,
                                                                 const int32_t* __restrict__ start,
                                                                 int ndesc) {
  __shared__ PushSmem<PartF32R, true> sm;
  const int item = (int)blockIdx.x;
  int lo = 0, hi = ndesc;  // start[lo] <= item < start[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (start[mid] <= item) lo = mid;
    else hi = mid;
  }
  const PIC_CONST PushDescF32* d = (const PIC_CONST PushDescF32*)(descs + lo);
  push_tile<true>(d, d->span * (int)xcd_interleave(item - start[lo], d->chunk), d->span, sm);
}

// ---------------------------------------------------------------- push, FP64
// The same kernel on FP64 records: positions in cell units, velocities in m/s;
// an empty slot has z = -1.  The field window holds (Ex,Ey),(Ez,0) pairs.
constexpr int kWinF64 = 1053;  // window capacity (nodes): a tile pair with a 2-cell margin
struct PushHot64 {
  int nx, ny, nz;
  double qm_dt, dt_dx;
};

template <bool kMove>
struct PushSmem<PartF64, kMove> {
  double2 E[kMove ? 2 * kWinF64 : 1];
  double rho[kWinF64];
  unsigned tally[TL_N];
  int ncoll, nout, far;
  CandStage<double, kMove ? kCandF64 : 1> cand;
};
template <bool kMove>
__device__ __forceinline__ void push_tile(const PIC_CONST PushDescF64* d, int tidx, int span,
                                          PushSmem<PartF64, kMove>& sm) {
  const int beg = d->L.tstart[tidx], end = d->L.tstart[tidx + span];
  if (kMove && threadIdx.x < span) {
    d->L.coll_cnt[tidx + threadIdx.x] = 0;
    d->L.out_cnt[tidx + threadIdx.x] = 0;
  }
  if (beg >= end) return;
  const PushHot64 S{d->S.nx, d->S.ny, d->S.nz, d->S.qm_dt, d->S.dt_dx};
  const Tile tile = make_tile(tidx, d->L, S.nx, S.ny, S.nz, d->S.margin, kWinF64, span);
  const int vol = tile.on ? tile.tx * tile.ty * tile.tz : 0;
  const float rtx = 1.0f / (float)max(tile.tx, 1), rtxy = 1.0f / (float)max(tile.tx * tile.ty, 1);
  for (int t = threadIdx.x; t < vol; t += kBlock) {
    if (kMove) {
      const long node = tile_node(tile, t, rtx, rtxy, S.nx, S.ny, d->S.nxy);
      sm.E[2 * t] = d->E[2 * node];
      sm.E[2 * t + 1] = d->E[2 * node + 1];
    }
    sm.rho[t] = 0.0;
  }
  if (threadIdx.x < TL_N) sm.tally[threadIdx.x] = 0;
  if (threadIdx.x == 0) {
    sm.ncoll = 0;
    sm.far = 0;
    sm.nout = 0;
  }
  const bool md_near = window_meets_md(tile, d->md, S.nx, S.ny);
  const PartF64 P = desc_records(d);
  int32_t* const coll = d->L.coll + beg;
  int32_t* const out = d->L.out + beg;
  const double vfast2 = d->S.vfast2, sign = d->S.sign;
  const uint32_t step = kMove ? *d->S.step : 0u, key0 = d->S.key0, key1 = d->S.key1, sp = (uint32_t)d->S.sp;
  const bool cand_on = d->S.T_null != 0;
  const uint32_t T_last = (uint32_t)(d->S.T_null - 1);
  __syncthreads();
  int n_fast = 0;
  for (int base = beg; base < end; base += kChunk) {
    const int p0 = base + kPPT * (int)threadIdx.x;
    const bool have = p0 < end;  // four slots in the tile, or none
    const long g4 = p0 / kPPT;
    double x[kPPT][3], v[kPPT][3];
    uint32_t id[kPPT] = {};
#pragma unroll
    for (int q = 0; q < kPPT; ++q) {
      x[q][0] = x[q][1] = v[q][0] = v[q][1] = v[q][2] = 0.0;
      x[q][2] = -1.0;
    }
    if (have) {
#define PIC_LOAD4(arr, dst, a)                                            \
  {                                                                       \
    const double2 lo = reinterpret_cast<const double2*>(arr)[2 * g4];     \
    const double2 hi = reinterpret_cast<const double2*>(arr)[2 * g4 + 1]; \
    dst[0][a] = lo.x;                                                     \
    dst[1][a] = lo.y;                                                     \
    dst[2][a] = hi.x;                                                     \
    dst[3][a] = hi.y;                                                     \
  }
      PIC_LOAD4(P.x, x, 0)
      PIC_LOAD4(P.y, x, 1)
      PIC_LOAD4(P.z, x, 2)
      PIC_LOAD4(P.vx, v, 0)
      PIC_LOAD4(P.vy, v, 1)
      PIC_LOAD4(P.vz, v, 2)
#undef PIC_LOAD4
      const uint4 I4 = reinterpret_cast<const uint4*>(P.id)[g4];
      id[0] = I4.x;
      id[1] = I4.y;
      id[2] = I4.z;
      id[3] = I4.w;
    }
    int cell[kPPT];
    unsigned st = 0, live = 0;  // as in the FP32R push
#pragma unroll
    for (int q = 0; q < kPPT; ++q) {
      const bool full = x[q][2] >= 0.0;
      const int i0 = (int)floor(x[q][0]), j0 = (int)floor(x[q][1]), k0 = (int)floor(x[q][2]);
      cell[q] = -1;
      if (!kMove) {
        if (full) {
          live |= 1u << q;
          cell[q] = pack_cell(i0, j0, k0);
        }
        continue;
      }
      const int lb = tile_cell(tile, i0, j0, k0, S.nx, S.ny);
      int e = !full ? ST_NONE : (lb < 0 ? ST_OUT : ST_ALIVE);
      if (full && (md_near || lb < 0) && push_in_md(d, pack_cell(i0, j0, k0))) e = ST_MD;
      if (e == ST_ALIVE) {
        double Ep[3];
        {
          const double fx = x[q][0] - i0, fy = x[q][1] - j0, fz = x[q][2] - k0;
          const double wx[2] = {1.0 - fx, fx}, wy[2] = {1.0 - fy, fy}, wz[2] = {1.0 - fz, fz};
          Ep[0] = Ep[1] = Ep[2] = 0.0;
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            const int l = lb + (t & 1) + tile.tx * (((t >> 1) & 1) + tile.ty * (t >> 2));
            const double w = wx[t & 1] * wy[(t >> 1) & 1] * wz[t >> 2];
            const double2 a = sm.E[2 * l], b2 = sm.E[2 * l + 1];
            Ep[0] += w * a.x;
            Ep[1] += w * a.y;
            Ep[2] += w * b2.x;
          }
        }
        e = push_one_f64(S, Ep, x[q], v[q]);
        n_fast += v[q][0] * v[q][0] + v[q][1] * v[q][1] + v[q][2] * v[q][2] >= vfast2;
        if (e == ST_ALIVE) {
          cell[q] = pack_cell((int)floor(x[q][0]), (int)floor(x[q][1]), (int)floor(x[q][2]));
          live |= 1u << q;
        } else {
          x[q][2] = -1.0;
        }
      }
      st |= (unsigned)e << (4 * q);
    }
    if (kMove) {
      if (cand_on) {
        uint32_t w0[kPPT], c0 = key0, c1 = key1;
        asm volatile("" : "+s"(c0), "+s"(c1));
        philox_word0<kPPT>(id, step, kColl, sp, c0, c1, w0);
        unsigned cm = 0;
#pragma unroll
        for (int q = 0; q < kPPT; ++q) cm |= (w0[q] <= T_last ? 1u : 0u) << q;
        cm &= live;
        if (__any(cm)) cand_append(cm, sm.cand, coll, &sm.ncoll, p0, id, v);
      }
      if (md_near && have) d->L.mask[g4] = 0;
      if (__any((st & 0xbbbbu) != 0u))
        push_events(st, p0, have, md_near, d->L, out, &sm.nout, sm.tally);
      if (have) {
#define PIC_STORE4(arr, srcv, a)                                                          \
  {                                                                                       \
    reinterpret_cast<double2*>(arr)[2 * g4] = make_double2(srcv[0][a], srcv[1][a]);     \
    reinterpret_cast<double2*>(arr)[2 * g4 + 1] = make_double2(srcv[2][a], srcv[3][a]); \
  }
        PIC_STORE4(P.x, x, 0)
        PIC_STORE4(P.y, x, 1)
        PIC_STORE4(P.z, x, 2)
        PIC_STORE4(P.vx, v, 0)
        PIC_STORE4(P.vy, v, 1)
        PIC_STORE4(P.vz, v, 2)
#undef PIC_STORE4
      }
    }

    double acc[8];
    int acc_cell = -1;
    auto flush = [&]() {
      const int ai = cell_i(acc_cell), aj = cell_j(acc_cell), ak = cell_k(acc_cell);
      const int lb = tile_cell(tile, ai, aj, ak, S.nx, S.ny);
      if (lb >= 0) {
#pragma unroll
        for (int t = 0; t < 8; ++t)
          atomicAdd(&sm.rho[lb + (t & 1) + tile.tx * (((t >> 1) & 1) + tile.ty * (t >> 2))], acc[t]);
        return;
      }
      if (kMove && push_in_md(d, acc_cell)) sm.far = 1;
      corner_add<double>(tile, -1, sm.rho, d->rho, d->S, ai, aj, ak, acc);
    };
#pragma unroll
    for (int q = 0; q < kPPT; ++q) {
      if (!((live >> q) & 1u)) continue;
      double w[8];
      const int i = cell_i(cell[q]), j = cell_j(cell[q]), k = cell_k(cell[q]);
      cic_weights_d(x[q][0] - i, x[q][1] - j, x[q][2] - k, sign, w);
      if (cell[q] == acc_cell) {
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[t] += w[t];
      } else {
        if (acc_cell >= 0) flush();
        acc_cell = cell[q];
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[t] = w[t];
      }
    }
    if (acc_cell >= 0) flush();
  }
  if (kMove) tally_add(sm.tally, TL_FAST, n_fast);
  __syncthreads();
  if constexpr (kMove) cand_collide(P, d->S, sm.cand, sm.ncoll, sm.tally);
  double* const rho = d->rho;
  const long nxy = d->S.nxy;
  const float qtx = 1.0f / (float)max(tile.tx, 1), qtxy = 1.0f / (float)max(tile.tx * tile.ty, 1);
  for (int t = threadIdx.x; t < vol; t += kBlock) {
    const double val = sm.rho[t];
    if (val != 0.0) unsafeAtomicAdd(&rho[tile_node(tile, t, qtx, qtxy, S.nx, S.ny, nxy)], val);
  }
  if (kMove) {
    if (threadIdx.x == 0) {
      d->L.coll_cnt[tidx] = max(0, sm.ncoll - kCandF64);
      d->L.out_cnt[tidx] = sm.nout;
    }
    __syncthreads();
    tally_store(sm.tally, d->L.tally + (long)TL_N * tidx);
    if (sm.far && !md_near) list_far(P, d->L, d->md, S.nx, S.ny, beg, end, sm.nout);
  }
}
// (at most 168 VGPRs: three waves per SIMD; 52 KB of LDS allow three blocks a CU)
template <bool kMove>
__global__ __launch_bounds__(kBlock, 3) void push_f64_kernel(const PushDescF64* descs, int nb,
                                                          int span, int chunk) {
  __shared__ PushSmem<PartF64, kMove> sm;
  const int sp = (int)blockIdx.x >= nb ? 1 : 0, b = (int)blockIdx.x - sp * nb;
  push_tile<kMove>((const PIC_CONST PushDescF64*)(descs + sp), span * (int)xcd_interleave(b, chunk), span, sm);
}

// ---------------------------------------------------------------- MD particles
// The particles that started the step inside an MD cube: the sub-cycled PPPM
// motion in FP64, grain and electrode absorption, the deposit (md_block); the
// lists kernel collides them.  Four lanes or one per entry of the dense list.
__device__ __forceinline__ void load_d(const PartF64& P, long p, double x[3], double v[3]) {
  x[0] = P.x[p];
  x[1] = P.y[p];
  x[2] = P.z[p];
  v[0] = P.vx[p];
  v[1] = P.vy[p];
  v[2] = P.vz[p];
}
__device__ __forceinline__ void load_d(const PartF32R& P, long p, double x[3], double v[3]) {
  const int c = P.cell[p];
  x[0] = (double)cell_i(c) + (double)P.ox[p];
  x[1] = (double)cell_j(c) + (double)P.oy[p];
  x[2] = (double)cell_k(c) + (double)P.oz[p];
  v[0] = P.vx[p];
  v[1] = P.vy[p];
  v[2] = P.vz[p];
}

// store the survivor; returns its cell (-1 if rounding put it on the rf
// electrode) and the eight corner shares of its charge
template <typename H>
__device__ __forceinline__ int store_d(const PartF64& P, long p, const double x[3],
                                       const double v[3], const H& S, double part[8]) {
  P.x[p] = x[0];
  P.y[p] = x[1];
  P.z[p] = x[2];
  P.vx[p] = v[0];
  P.vy[p] = v[1];
  P.vz[p] = v[2];
  const int i = (int)floor(x[0]), j = (int)floor(x[1]), k = (int)floor(x[2]);
  cic_weights_d(x[0] - i, x[1] - j, x[2] - k, S.sign, part);
  return pack_cell(i, j, k);
}
template <typename H>
__device__ __forceinline__ int store_d(const PartF32R& P, long p, const double x[3],
                                       const double v[3], const H& S,
                                       long long part[8]) {
  int c[3];
  float f[3];
  const int n3[3] = {S.nx, S.ny, S.nz};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    c[a] = (int)floor(x[a]);
    f[a] = (float)(x[a] - (double)c[a]);
    if (f[a] >= 1.0f) {
      f[a] = 0.0f;
      c[a] += 1;
      if (a < 2 && c[a] == n3[a]) c[a] = 0;
    }
  }
  P.vx[p] = (float)v[0];
  P.vy[p] = (float)v[1];
  P.vz[p] = (float)v[2];
  if (c[2] >= S.nz) {
    P.cell[p] = -1;
    return -1;
  }
  P.cell[p] = pack_cell(c[0], c[1], c[2]);
  P.ox[p] = f[0];
  P.oy[p] = f[1];
  P.oz[p] = f[2];
  split8(S.Qp, f[0], f[1], f[2], part);
#pragma unroll
  for (int t = 0; t < 8; ++t) part[t] *= S.isign;
  return P.cell[p];
}

template <typename T>
__device__ __forceinline__ T wave_sum_t(T v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// The charges of a wave's MD particles to the global mesh.  The particles of
// a cell of the dense list tend to sit in neighbouring lanes and hit the same
// eight nodes, which all MD blocks share, so the wave first sums the corner
// shares of each of its first kDepGroups distinct cells in LDS (for the
// fixed-point charge the sums are exact and the mesh does not depend on the
// grouping); the remaining lanes add their own shares.
constexpr int kDepGroups = 16;
// what the wave's lanes wrote to LDS is seen by all of them
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
template <typename A>
__device__ __forceinline__ void deposit_wave(A (*s_sum)[8], int* s_cell, A* __restrict__ rho,
                                             const SpeciesStep& S, int cell, const A part[8]) {
  const int lane = threadIdx.x & 63;
  unsigned long long pending = __ballot(cell >= 0);
  int mine = -1, n = 0;
  for (; n < kDepGroups && pending; ++n) {
    const int key = __shfl(cell, __ffsll((long long)pending) - 1, 64);
    if (cell == key) mine = n;
    if (lane == 0) s_cell[n] = key;
    pending &= ~__ballot(cell == key);
  }
  for (int t = lane; t < 8 * n; t += 64) (&s_sum[0][0])[t] = (A)0;
  wave_sync();
  if (mine >= 0) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      if constexpr (std::is_same<A, long long>::value)
        atomicAdd((unsigned long long*)&s_sum[mine][t], (unsigned long long)part[t]);
      else
        atomicAdd(&s_sum[mine][t], part[t]);
    }
  }
  wave_sync();
  for (int e = lane; e < 8 * n; e += 64) {
    const int c = s_cell[e >> 3], t = e & 7;
    int i = cell_i(c) + (t & 1), j = cell_j(c) + ((t >> 1) & 1);
    if (i == S.nx) i = 0;
    if (j == S.ny) j = 0;
    atomic_add_acc(&rho[i + (long)S.nx * j + (long)S.nxy * (cell_k(c) + (t >> 2))], (&s_sum[0][0])[e]);
  }
  Tile none{};
  if (cell >= 0 && mine < 0)
    corner_add<A>(none, -1, nullptr, rho, S, cell_i(cell), cell_j(cell), cell_k(cell), part);
  wave_sync();  // the sums are free again
}

__device__ __forceinline__ void kill(const PartF64& P, long p) { P.z[p] = -1.0; }
__device__ __forceinline__ void kill(const PartF32R& P, long p) { P.cell[p] = -1; }
// slot p of src into slot p of dst (an empty src slot empties dst's)
__device__ __forceinline__ void copy_rec(const PartF64& src, const PartF64& dst, long p) {
  const double a = src.x[p], b = src.y[p], c = src.z[p], f = src.vx[p], g = src.vy[p], h = src.vz[p];
  dst.x[p] = a;
  dst.y[p] = b;
  dst.z[p] = c;
  dst.vx[p] = f;
  dst.vy[p] = g;
  dst.vz[p] = h;
}
__device__ __forceinline__ void copy_rec(const PartF32R& src, const PartF32R& dst, long p) {
  // (every load before the first store: one memory round trip)
  const int c = src.cell[p];
  const float a = src.ox[p], b = src.oy[p], e = src.oz[p], f = src.vx[p], g = src.vy[p], h = src.vz[p];
  dst.cell[p] = c;
  if (c < 0) return;
  dst.ox[p] = a;
  dst.oy[p] = b;
  dst.oz[p] = e;
  dst.vx[p] = f;
  dst.vy[p] = g;
  dst.vz[p] = h;
}

// The MD particles of the dense list of this step, a wave a group of them, in
// blocks of kWaves waves: blocks [0, pr.nb) the electrons', [pr.nb, 2 pr.nb) the
// ions'; events go to the wave's own tally row, grain hits to LDS counters
// first.  The particles are read from P and their new states written to the same
// slots of D, the species' other record buffer, so that this runs beside the
// push; the lists kernel after both copies the states back and takes the
// survivors' collisions (here they cost more registers: 113 us became 147 in the
// 64x64x256 box).
constexpr int kMdThreads = 64;
// lists up to this length move four lanes a particle (about the particles that
// one lane each would leave the chip's 1,024 SIMDs a wave or less)
constexpr int kMdQuad = 49152;
constexpr int kMdStage = 256;  // grains staged in LDS
template <typename RT, int kWaves>
struct MdSmem {
  RT sum[kWaves][kDepGroups][8];
  double gpos[3 * kMdStage], Qc[kMdStage];
  unsigned hits[kMdStage];
  int cell[kWaves][kDepGroups];
};
template <int kWaves, typename PT, typename ET, typename RT>
__device__ __forceinline__ void md_block(const SpeciesPair<PT>& pr, const PT& D0, const PT& D1,
                                         const ET* __restrict__ E, RT* __restrict__ rho,
                                         const MdTables& md,
                                         unsigned long long* __restrict__ grain_count, int block,
                                         MdSmem<RT, kWaves>& sm) {
  const int sp = block >= pr.nb;
  const PT P = pr.P[sp];
  const PT D = sp ? D1 : D0;
  const SpeciesStep S = pr.S[sp];
  const WorkLists L = pr.L[sp];
  const int total = *L.n_md;
  const int per = total <= kMdQuad ? 16 : 64;  // particles a wave takes at a time
  const int b0 = (block - sp * pr.nb) * kWaves;
  if ((long)b0 * per >= total) return;
  const int lane = (int)threadIdx.x & 63;
  const int wave = kWaves == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int bid = b0 + wave, nw = pr.nb * kWaves;
  const bool staged = md.n_grains <= kMdStage;
  for (int t = threadIdx.x; t < min(md.n_grains, kMdStage); t += 64 * kWaves) {
    sm.hits[t] = 0u;
    if (staged) {
      sm.Qc[t] = md.Q[t] * S.coul_c;
      double gx = md.gpos[3 * t] - md.bx0, gy = md.gpos[3 * t + 1] - md.by0;
      sm.gpos[3 * t] = gx < 0.0 ? gx + S.nx : gx;
      sm.gpos[3 * t + 1] = gy < 0.0 ? gy + S.ny : gy;
      sm.gpos[3 * t + 2] = md.gpos[3 * t + 2];
    }
  }
  __syncthreads();
  const GrainView G{(LdsDoubles)sm.gpos, (LdsDoubles)sm.Qc, !staged};
  const double a2_cells = md.a2 / (S.dx * S.dx);
  const bool image = md.bsx == S.nx || md.bsy == S.ny;
  int n_w0 = 0, n_w1 = 0, n_bad = 0, n_dead = 0;
  auto move = [&](auto lanes, long idx, int sub_lane) {
    int st = ST_NONE, cell = -1;
    RT part[8];
    if (idx < total) {
      const long p = L.md[idx];
      double x[3], v[3];
      load_d(P, p, x, v);
      x[0] -= md.bx0;
      x[1] -= md.by0;
      if (x[0] < 0.0) x[0] = wrap_coord(x[0], S.nx);
      if (x[1] < 0.0) x[1] = wrap_coord(x[1], S.ny);
      int hit = -1;
      st = md_move<decltype(lanes)::value>(E, md, G, S, a2_cells, image, x, v, hit);
      if (sub_lane != 0) {
        st = ST_NONE;  // (the quad's first lane settles the particle)
      } else if (st == ST_ALIVE) {
        x[0] = wrap_coord(x[0] + md.bx0, S.nx);
        x[1] = wrap_coord(x[1] + md.by0, S.ny);
        cell = store_d(D, p, x, v, S, part);
        if (cell < 0) st = ST_WALL1;
      } else {
        if (st == ST_GRAIN) {
          if (hit < kMdStage) atomicAdd(&sm.hits[hit], 1u);
          else atomicAdd(&grain_count[2 * hit + S.sp], 1ull);
        }
        kill(D, p);
      }
    }
    deposit_wave<RT>(sm.sum[wave], sm.cell[wave], rho, S, cell, part);
    n_w0 += st == ST_WALL0;
    n_w1 += st == ST_WALL1;
    n_bad += st == ST_BAD;
    n_dead += st == ST_WALL0 || st == ST_WALL1 || st == ST_BAD || st == ST_GRAIN;
  };
  if (total <= kMdQuad) {
    for (long base = (long)bid * 16; base < total; base += (long)nw * 16)
      move(std::integral_constant<int, 4>{}, base + (lane >> 2), lane & 3);
  } else {
    for (long base = (long)bid * 64; base < total; base += (long)nw * 64)
      move(std::integral_constant<int, 1>{}, base + lane, 0);
  }
  int c4[4] = {n_w0, n_w1, n_bad, n_dead};
#pragma unroll
  for (int k = 0; k < 4; ++k) c4[k] = wave_sum(c4[k]);
  if (lane == 0) {  // this wave's own tally row (no atomics)
    unsigned long long* tally = L.tally + (long)TL_N * (L.ngrid + bid);
    const int kinds[4] = {TL_W0, TL_W1, TL_BAD, TL_DEAD};
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (c4[k]) tally[kinds[k]] += (unsigned long long)c4[k];
  }
  __syncthreads();
  for (int t = threadIdx.x; t < min(md.n_grains, kMdStage); t += 64 * kWaves)
    if (sm.hits[t]) atomicAdd(&grain_count[2 * t + S.sp], (unsigned long long)sm.hits[t]);
}
template <typename PT, typename ET, typename RT>
__global__ __launch_bounds__(kMdThreads) void md_kernel(SpeciesPair<PT> pr, PT D0, PT D1,
                                                        const ET* __restrict__ E,
                                                        RT* __restrict__ rho, MdTables md,
                                                        unsigned long long* __restrict__ grain_count) {
  __shared__ MdSmem<RT, 1> sm;
  md_block<1>(pr, D0, D1, E, rho, md, grain_count, (int)blockIdx.x, sm);
}

// The push and the MD particles' motion in one launch, the MD blocks (four waves
// each) first, for a box whose blocks are all resident at once: a second stream
// for the MD kernel costs a fork and a join, about 5 us each (16x16x32 cells: from
// the fields to the lists 44 us with two launches, 34 us so, before the chain of
// md_move was shortened to 28).  A larger box keeps two:
// the MD motion's registers (two waves per SIMD) would be the push's too.
template <typename PT, typename Desc, typename ET, typename RT>
__global__ __launch_bounds__(kBlock, 2) void push_md_kernel(const Desc* descs, int nb, int span,
                                                         int chunk, SpeciesPair<PT> pr, PT D0,
                                                         PT D1, const ET* __restrict__ E,
                                                         RT* __restrict__ rho, MdTables md,
                                                         unsigned long long* __restrict__ grain_count) {
  __shared__ union {
    PushSmem<PT, true> push;
    MdSmem<RT, kBlock / 64> md;
  } sm;
  const int block = (int)blockIdx.x - 2 * pr.nb;
  if (block < 0) {
    md_block<kBlock / 64>(pr, D0, D1, E, rho, md, grain_count, (int)blockIdx.x, sm.md);
    return;
  }
  const int sp = block >= nb ? 1 : 0;
  push_tile<true>((const PIC_CONST Desc*)(descs + sp), span * (int)xcd_interleave(block - sp * nb, chunk), span,
                  sm.push);
}

// ---------------------------------------------------------------- moments
// Density and flux moments of one species on the mesh nodes (the densities
// and fluxes of Sec. IV): per node the sums over the particles of W and of
// v W, where W is the particle's CIC weight for the node, the same
// assignment as the charge deposit of Sec. III.  The host scales them by
// w / dx^3.  v is the stored half-step velocity v_{k-1/2}.  mom is [4][nn]:
// W, v_x W, v_y W, v_z W.  For the time averages (avg.step non-null) the sums
// go to the rf-phase bin of the current step, avg.stride doubles further per
// bin.
//
// One block per tile.  Per cell the sums are a 4 x n by n x 8 product, (1, v)
// of its n particles by their weights, and go through the FP64 matrix units
// (the 4x4x4 form on four cells at a time, two instructions for the eight
// corners), so a cell's particles have to lie side by side: a chunk of the
// tile's slots is read once, coalesced, and counted, ranked and stored by cell in
// LDS (the particles have drifted since the last re-binning).  The four cells of a
// wave take as many rounds as the fullest, so the tile's own cells, all about
// as full, come first and the drift margin's after them.  The cells' sums meet
// in a window of the tile's nodes plus the margin (at most 2 cells) and reach
// the mesh once; a particle outside the window adds to the mesh directly.
// One thread a run of slots with 32 sums in registers was bound by its LDS
// atomics: 32 a run, and a run ends wherever a particle has drifted.  Now vector
// instructions take 44 to 52 % of the issue slots, and a wave waits 55 to 58 % of
// its time (counters: memory, LDS and barriers are not told apart).
// 64x64x256 cells, 32 per cell, mean of the species: FP32R 733 us -> 445 (0.94 GB),
// FP64 1326 -> 558 (1.6 GB); 128x128x512, 16 per cell, FP32R 2,850 -> 2,240 (3.8 GB).
constexpr int kMomWin = 729;  // most nodes of a window
// slots of a chunk, with LDS for two blocks a CU at the largest window: a tile of
// 32 per cell in FP32R, half of one in FP64; and, for a tile of 16 in FP32R, half
// of that, of which a margin of one cell leaves room for four blocks of 256
// threads (128x128x512 cells, 16 per cell: 1.55 ms against 2.15 in 512) and one
// of two cells room for two, of 512 threads (2.9 ms against 3.5 in 256)
constexpr int kMomCapFull = 2160, kMomCapHalf = 1080;
__host__ __device__ constexpr size_t mom_lds(int nodes, int cap, size_t v) {
  return nodes * 32 + cap * 6 * v + (64 + nodes + 1) * 8;
}
// a slot's cell (i, j, k), offsets in the cell and velocity; false if it is free
__device__ __forceinline__ bool mom_load(const PartF32R& P, long p, int c[3], float r[6]) {
  const int cell = P.cell[p];
  r[0] = P.ox[p];
  r[1] = P.oy[p];
  r[2] = P.oz[p];
  r[3] = P.vx[p];
  r[4] = P.vy[p];
  r[5] = P.vz[p];
  c[0] = cell_i(cell);
  c[1] = cell_j(cell);
  c[2] = cell_k(cell);
  return cell >= 0;
}
__device__ __forceinline__ bool mom_load(const PartF64& P, long p, int c[3], double r[6]) {
  double x[3];
  load_d(P, p, x, r + 3);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double f = floor(x[a]);
    c[a] = (int)f;
    r[a] = x[a] - f;
  }
  return x[2] >= 0.0;
}

// inclusive sums over the wave
__device__ __forceinline__ int wave_prefix(int v) {
  const int lane = (int)threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(v, d, 64);
    if (lane >= d) v += o;
  }
  return v;
}

// grid (tiles along x, along y, along z and the grid's padding), mom_lds() bytes of LDS
template <typename PT, int kT, int kCap>
__global__ __launch_bounds__(kT, 4) void moments_kernel(PT P, SpeciesStep S, WorkLists L,
                                                                 double* __restrict__ mom, long nn,
                                                                 AvgBins avg, int nodes) {
  using V = typename VelOf<PT>::type;
  constexpr int kPer = (kCap + kT - 1) / kT, kWaves = kT / 64;
  constexpr int kIds = (64 + kMomWin + kT - 1) / kT;  // ids a thread of the scan, at most
  extern __shared__ double s_dyn[];
  double* s_m = s_dyn;                           // [4][nodes]
  V* s_r = (V*)(s_m + 4 * nodes);                // [6][kCap] offsets and velocities, by cell
  const int ids = 64 + nodes;                    // cell ids: the tile's own, then by window node
  int* s_start = (int*)(s_r + 6 * kCap);         // [ids] particles per cell id, then first entry
  uint32_t* s_list = (uint32_t*)(s_start + ids + 1);  // the occupied cells: first entry << 16 | node
  __shared__ int s_wave[kWaves];
  const int tid = (int)threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ti = blockIdx.x, tj = blockIdx.y, tk = blockIdx.z;
  const int t = (tk * L.nty + tj) * L.ntx + ti;
  if (t >= L.ngrid) return;
  const int a = L.tstart[t], b = L.tstart[t + 1];
  if (a == b) return;
  if (avg.step) mom += avg.stride * phase_bin(*avg.step, avg.f_rf, avg.dt, avg.nbins);
  Tile T{};
  if (tk < L.ntz) T = tile_window(ti, tj, tk, S.nx, S.ny, S.nz, S.margin, nodes, 1);
  // the tile's own cells in window cells
  const int wx = 4 * ti - T.x0, wy = 4 * tj - T.y0, wz = 4 * tk - T.k0;
  for (int u = tid; u < 4 * nodes; u += kT) s_m[u] = 0.0;
  const int chunks = (b - a + kCap - 1) / kCap, per = (b - a + chunks - 1) / chunks;
  for (int p0 = a; p0 < b; p0 += per) {
    const int n = min(per, b - p0);
    for (int u = tid; u < ids; u += kT) s_start[u] = 0;
    __syncthreads();
    V r[kPer][6];
    int id[kPer], rank[kPer], far = 0;
#pragma unroll
    for (int m = 0; m < kPer; ++m) {
      const int u = tid + m * kT;
      id[m] = -1;
      rank[m] = 0;
      if (u >= n) continue;
      int c[3];
      if (!mom_load(P, p0 + u, c, r[m])) continue;
      const int lb = tile_cell(T, c[0], c[1], c[2], S.nx, S.ny);
      if (lb < 0) {
        far |= 1 << m;
        continue;
      }
      const int li = c[0] - 4 * ti, lj = c[1] - 4 * tj, lk = c[2] - 4 * tk;
      id[m] = ((li | lj | lk) & ~3) == 0 ? (lk * 4 + lj) * 4 + li : 64 + lb;
      rank[m] = atomicAdd(&s_start[id[m]], 1);
    }
    // outside the window: straight to the mesh
    for (; far; far &= far - 1) {
      int c[3];
      V q[6];
      mom_load(P, p0 + tid + (__ffs(far) - 1) * kT, c, q);
      double w[8], val[8];
      cic_weights_d(q[0], q[1], q[2], 1.0, w);
      corner_add<double>(T, -1, nullptr, mom, S, c[0], c[1], c[2], w);
#pragma unroll
      for (int d = 0; d < 3; ++d) {
#pragma unroll
        for (int e = 0; e < 8; ++e) val[e] = (double)q[3 + d] * w[e];
        corner_add<double>(T, -1, nullptr, mom + (d + 1) * nn, S, c[0], c[1], c[2], val);
      }
    }
    __syncthreads();
    // first entries and the list of occupied cells: one scan of both counts
    int cnt[kIds], own = 0, sum = 0;
    if (64 * kIds * wave < ids) {
#pragma unroll
      for (int i = 0; i < kIds; ++i) {
        cnt[i] = kIds * tid + i < ids ? s_start[kIds * tid + i] : 0;
        own += cnt[i] + (cnt[i] ? 1 << 16 : 0);
      }
      sum = wave_prefix(own);
    }
    if (lane == 63) s_wave[wave] = sum;
    __syncthreads();
    int before = sum - own, all = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      if (w < wave) before += s_wave[w];
      all += s_wave[w];
    }
    const int ncell = all >> 16;
    if (64 * kIds * wave < ids) {
#pragma unroll
      for (int i = 0; i < kIds; ++i) {
        const int c = kIds * tid + i;
        if (c < ids) s_start[c] = before & 0xffff;
        if (cnt[i]) {
          const int node = c >= 64 ? c - 64 : ((wz + (c >> 4)) * T.ty + wy + ((c >> 2) & 3)) * T.tx + wx + (c & 3);
          s_list[before >> 16] = (uint32_t)before << 16 | (uint32_t)node;
          before += cnt[i] + (1 << 16);
        }
      }
    }
    if (tid == 0) s_list[ncell] = (uint32_t)all << 16;
    __syncthreads();
#pragma unroll
    for (int m = 0; m < kPer; ++m) {
      if (id[m] < 0) continue;
      const int e = s_start[id[m]] + rank[m];
#pragma unroll
      for (int q = 0; q < 6; ++q) s_r[q * kCap + e] = r[m][q];
    }
    __syncthreads();
    // lane = j + 4 cell + 16 k: operand A (quantity j, particle k), operand B (particle
    // k, corner j), result (quantity k, corner j)
    const int j = lane & 3, cell = (lane >> 2) & 3, k = lane >> 4;
    const double ax = j & 1 ? 0.0 : 1.0, bx = j & 1 ? 1.0 : -1.0;
    const double ay = j & 2 ? 0.0 : 1.0, by = j & 2 ? 1.0 : -1.0;
    const V* vel = s_r + (j ? 2 + j : 3) * kCap;
    double* out = s_m + k * nodes + (j & 1) + T.tx * (j >> 1);
    for (int g = 4 * wave; g < ncell; g += 4 * kWaves) {
      const int at = min(g + cell, ncell - 1);
      const bool have = g + cell < ncell;
      const uint32_t c = s_list[at];
      const int s = (int)(c >> 16), e = have ? (int)(s_list[at + 1] >> 16) : s;
      // the matrix instructions take all lanes: as many rounds as the fullest cell
      // of the four needs.  The count has to stay a scalar: the sums then stay in
      // their registers from the first round to the last (with the loop left on a
      // ballot the compiler copied a result at the loop's head without the wait
      // states it needs, and the sums came out wrong)
      int most = e - s;
      most = max(most, __builtin_amdgcn_update_dpp(0, most, 0x124, 0xf, 0xf, false));  // row_ror:4
      most = max(most, __builtin_amdgcn_update_dpp(0, most, 0x128, 0xf, 0xf, false));  // row_ror:8
      most = __builtin_amdgcn_readfirstlane(most);
      double lo = 0.0, hi = 0.0;
      for (int u = 0; u < most; u += 4) {
        const bool in = s + u + k < e;
        const int p = in ? s + u + k : s;
        const double fx = s_r[p], fy = s_r[kCap + p], fz = s_r[2 * kCap + p];
        const V v = vel[p];
        const double A = in ? (j ? (double)v : 1.0) : 0.0;
        const double w = (ax + bx * fx) * (ay + by * fy);
        lo = __builtin_amdgcn_mfma_f64_4x4x4f64(A, w * (1.0 - fz), lo, 0, 0, 0);
        hi = __builtin_amdgcn_mfma_f64_4x4x4f64(A, w * fz, hi, 0, 0, 0);
      }
      // the last results' wait states before anything that follows this statement.
      // It does not cover a copy placed between the last matrix instruction and
      // here; with the scalar count there is none
      asm volatile("s_nop 7\n\ts_nop 3" : "+v"(lo), "+v"(hi));
      if (have) {
        atomicAdd(&out[c & 0xffff], lo);
        atomicAdd(&out[(c & 0xffff) + T.tx * T.ty], hi);
      }
    }
    __syncthreads();
  }
  if (!T.on) return;
  const int nt = T.tx * T.ty * T.tz;
  const float rtx = 1.0f / (float)T.tx, rtxy = 1.0f / (float)(T.tx * T.ty);
  for (int u = tid; u < nt; u += kT) {
    const long node = tile_node(T, u, rtx, rtxy, S.nx, S.ny, S.nxy);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double sum = s_m[q * nodes + u];
      if (sum != 0.0) unsafeAtomicAdd(&mom[q * nn + node], sum);
    }
  }
}

// Fine diagnostic grid (the grid finer than the PIC cells over the grains'
// region, Sec. IV): a particle whose u = (x - o) / h lies in [0, m) on every
// axis adds its cloud-in-cell weights W and v W to the 8 nodes of its fine
// cell.  Grid-stride over the slots in use; the PIC cell is tested first, so
// the records of particles far from the box are not read whole.  Global FP64
// atomics: the box holds few particles per fine cell.
__device__ __forceinline__ bool fine_cell_near(const FineBox& fb, int i, int j, int k) {
  return i >= fb.lo[0] && i < fb.hi[0] && j >= fb.lo[1] && j < fb.hi[1] && k >= fb.lo[2] &&
         k < fb.hi[2];
}
__device__ __forceinline__ bool fine_near(const PartF64& P, long p, const FineBox& fb) {
  const double z = P.z[p];
  if (!(z >= 0.0)) return false;
  return fine_cell_near(fb, (int)floor(P.x[p]), (int)floor(P.y[p]), (int)floor(z));
}
__device__ __forceinline__ bool fine_near(const PartF32R& P, long p, const FineBox& fb) {
  const int c = P.cell[p];
  return c >= 0 && fine_cell_near(fb, cell_i(c), cell_j(c), cell_k(c));
}

// Both species in one launch (blockIdx.y): each alone waits mostly for its reads.
template <typename PT>
__global__ __launch_bounds__(256) void fine_moments_kernel(PT P0, PT P1, const int32_t* end0,
                                                           const int32_t* end1, FineBox fb,
                                                           double* __restrict__ mom,
                                                           AvgBins avg) {
  const PT P = blockIdx.y ? P1 : P0;
  const long total = blockIdx.y ? *end1 : *end0;
  if (avg.step) mom += avg.stride * phase_bin(*avg.step, avg.f_rf, avg.dt, avg.nbins);
  mom += 4 * fb.fn * blockIdx.y;
  for (long p = (long)blockIdx.x * blockDim.x + threadIdx.x; p < total;
       p += (long)gridDim.x * blockDim.x) {
    if (!fine_near(P, p, fb)) continue;
    double x[3], v[3], u[3];
    load_d(P, p, x, v);
    bool in = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      u[a] = (x[a] - fb.o[a]) / fb.h;
      in = in && u[a] >= 0.0 && u[a] < (double)fb.m[a];
    }
    if (!in) continue;
    const long i = (long)floor(u[0]), j = (long)floor(u[1]), k = (long)floor(u[2]);
    const double fx = u[0] - (double)i, fy = u[1] - (double)j, fz = u[2] - (double)k;
    const long base = (k * fb.my + j) * fb.mx + i;
#pragma unroll
    for (int cc = 0; cc < 2; ++cc)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          const double wt = (a ? fx : 1.0 - fx) * (b ? fy : 1.0 - fy) * (cc ? fz : 1.0 - fz);
          const long node = base + ((long)cc * fb.my + b) * fb.mx + a;
          unsafeAtomicAdd(&mom[node], wt);
#pragma unroll
          for (int q = 0; q < 3; ++q) unsafeAtomicAdd(&mom[(q + 1) * fb.fn + node], v[q] * wt);
        }
  }
}


// The MD particles' new states copied back from D and the collisions of those
// that survived, from their stored velocities (same list and tally rows as
// md_kernel, nb blocks of 64 threads).
template <typename PT, typename Desc>
__device__ __forceinline__ void md_collide_block(const PIC_CONST Desc* d, const PT& D, int bid,
                                                 int nb, int mcc) {
  const PT P = desc_records(d);
  const auto& S = d->S;
  const auto& L = d->L;
  const int total = *L.n_md;
  if ((long)bid * kMdThreads >= total) return;
  int n_coll = 0, n_cap = 0;
  for (int idx = bid * kMdThreads + (int)threadIdx.x; idx < total; idx += nb * kMdThreads) {
    const int p = L.md[idx];
    copy_rec(D, P, p);  // the sub-cycled kernel's result
    if (!mcc || !slot_alive(D, p)) continue;
    bool coll = false, capv = false;
    typename VelOf<PT>::type v[3] = {D.vx[p], D.vy[p], D.vz[p]};
    collide(S, P.id[p], v, coll, capv, p);
    if (coll) {
      P.vx[p] = v[0];
      P.vy[p] = v[1];
      P.vz[p] = v[2];
    }
    n_coll += coll;
    n_cap += capv;
  }
  n_coll = wave_sum(n_coll);
  n_cap = wave_sum(n_cap);
  if (threadIdx.x == 0) {
    unsigned long long* tally = L.tally + (long)TL_N * (L.ngrid + bid);
    if (n_coll) tally[TL_COLL] += (unsigned long long)n_coll;
    if (n_cap) tally[TL_CAP] += (unsigned long long)n_cap;
  }
}

// One wave takes kNearSlots slots of a push block near the MD cubes and lists
// those that are now in a cube for the next step, in slot order, with one
// reservation (the MD particles by their state in D, which other blocks copy
// back meanwhile; the particles outside the window list themselves,
// outlier_block).  Four slots a lane: the loads, the tables and the reservation
// depend on each other, and a wave that went through 1,024 slots in turn took
// four times that chain (16x16x32 cells: lists kernel 23 us, 7.4 us so).
constexpr int kNearSlots = 256;
template <typename PT, typename Desc>
__device__ __forceinline__ void near_block(const PIC_CONST Desc* d, const PT& D, int chunk,
                                           int chunks) {
  const PT P = desc_records(d);
  const auto& L = d->L;
  const auto& md = d->md;
  const int nx = d->S.nx, ny = d->S.ny;
  const int t0 = L.near[chunk / chunks];
  const int first = L.tstart[t0], end = L.tstart[t0 + d->span];
  const int lane = (int)threadIdx.x & 63;
  // (a push block with more slots than its chunks cover: the chunks take turns)
  for (int base = first + (chunk % chunks) * kNearSlots; base < end; base += chunks * kNearSlots) {
    const int p0 = base + 4 * lane;
    const unsigned m = p0 < end ? L.mask[p0 >> 2] : 0xf0u;
    bool in[4];
    int cnt = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int p = p0 + q;
      const bool moved = (m >> q) & 1u;
      in[q] = !(m & (16u << q)) && (moved ? slot_alive(D, p) : slot_alive(P, p)) &&
              in_md(md, nx, ny, moved ? slot_cell(D, p) : slot_cell(P, p));
      cnt += in[q];
    }
    int incl = cnt;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int t = __shfl_up(incl, off, 64);
      if (lane >= off) incl += t;
    }
    const int total = __shfl(incl, 63, 64);
    if (total == 0) continue;
    int at = 0;
    if (lane == 0) at = atomicAdd(L.n_md_next, total);
    at = __shfl(at, 0, 64) + incl - cnt;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (in[q]) L.md_next[at++] = p0 + q;
  }
}

// ---------------------------------------------------------------- packed lists
// One wave takes the list segments of `group` consecutive push blocks (at most
// 64) end to end: lane j holds segment j's place, and entry i of the whole lies
// in the segment found among the lanes.  A wave per segment instead left most
// lanes idle and a chain of dependent loads per push block (an ion block has
// one candidate or none): 64x64x256 75 us after the pushes, 128x128x512 950 us.
struct Segments {
  int start, end;  // of this lane's segment in the whole
  long first;      // its first slot in the list array
  int total;       // (wave-uniform)
};
__device__ __forceinline__ Segments segments(const int32_t* cnt, const int32_t* tstart, int block0,
                                             int nblocks, int span) {
  const int lane = (int)threadIdx.x & 63;
  Segments s;
  const bool on = lane < nblocks;
  const int t = (block0 + (on ? lane : 0)) * span;
  const int n = on ? cnt[t] : 0;
  s.first = tstart[t];
  int incl = n;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int v = __shfl_up(incl, off, 64);
    if (lane >= off) incl += v;
  }
  s.start = incl - n;
  s.end = incl;
  s.total = __shfl(incl, 63, 64);
  return s;
}
// the list entry i (< s.total, or any lane's spare call) of the segments
__device__ __forceinline__ int segment_entry(const Segments& s, const int32_t* list, int i) {
  int j = 0;  // the segments that end at or before entry i
#pragma unroll
  for (int step = 32; step > 0; step >>= 1)
    if (__shfl(s.end, j + step - 1, 64) <= i) j += step;
  const long first = __shfl(s.first, j & 63, 64);
  const int start = __shfl(s.start, j & 63, 64);
  return i < s.total ? list[first + (i - start)] : 0;
}

// ---------------------------------------------------------------- outliers
// Particles that started outside their push block's window (they drifted since
// the last sort): the same push with the field gathered from global memory and the
// charge deposited with global atomics, the collision done in place.  One wave
// takes the packed segments of a group of push blocks.
template <typename WL>
__device__ __forceinline__ void outlier_tally(const WL& L, int tidx, int w0, int w1, int bad,
                                              int coll, int cap, int fast) {
  w0 = wave_sum(w0);
  w1 = wave_sum(w1);
  bad = wave_sum(bad);
  coll = wave_sum(coll);
  cap = wave_sum(cap);
  fast = wave_sum(fast);
  if (threadIdx.x != 0) return;
  unsigned long long* tl = L.tally + (long)TL_N * tidx;
  tl[TL_W0] += w0;
  tl[TL_W1] += w1;
  tl[TL_BAD] += bad;
  tl[TL_COLL] += coll;
  tl[TL_CAP] += cap;
  tl[TL_DEAD] += w0 + w1 + bad;
  tl[TL_FAST] += fast;
}
// the outliers of `nblocks` push blocks from block0 of species sp
__device__ __forceinline__ void outlier_block(const PIC_CONST PushDescF32* d, const PartF32R& D, int do_mcc,
                                              int block0, int nblocks) {
  const PartF32R P = desc_records(d);
  const auto& S = d->S;
  const auto& L = d->L;
  const auto& md = d->md;
  const float4* __restrict__ E = d->E;
  long long* __restrict__ rho = d->rho;
  const Segments sg = segments(L.out_cnt, L.tstart, block0, nblocks, d->span);
  if (sg.total == 0) return;
  int t_w0 = 0, t_w1 = 0, t_bad = 0, t_coll = 0, t_cap = 0, t_fast = 0;
  for (int base = 0; base < sg.total; base += 64) {
    const int idx = base + (int)threadIdx.x;
    bool enters = false;
    int p = segment_entry(sg, L.out, idx);
    if (idx < sg.total && p < 0) {
      p = ~p;
      enters = slot_alive(D, p) && in_md(md, S.nx, S.ny, slot_cell(D, p));
    } else if (idx < sg.total) {
      const int c = P.cell[p];
      int ci = cell_i(c), cj = cell_j(c), ck = cell_k(c);
      float o[3] = {P.ox[p], P.oy[p], P.oz[p]};
      float v[3] = {P.vx[p], P.vy[p], P.vz[p]};
      float ec[8][3];
      const int i1 = ci + 1 == S.nx ? 0 : ci + 1;
      const int j1 = cj + 1 == S.ny ? 0 : cj + 1;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const float4 e = E[((t & 1) ? i1 : ci) + (long)S.nx * (((t >> 1) & 1) ? j1 : cj) +
                           (long)S.nxy * (ck + (t >> 2))];
        ec[t][0] = e.x;
        ec[t][1] = e.y;
        ec[t][2] = e.z;
      }
      const int st = push_one_f32(S, ec, o, v, ci, cj, ck);
      t_fast += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] >= S.vfast2_f;
      if (st == ST_ALIVE) {
        bool coll = false, capv = false;
        if (do_mcc) {
          const uint32_t id = P.id[p];
          const uint4 r = philox4x32_10(id, *S.step, kColl, (uint32_t)S.sp, S.key0, S.key1);
          if ((uint64_t)r.x < S.T_null) collide(S, id, v, coll, capv, p);
        }
        t_coll += coll;
        t_cap += capv;
        const int cn = pack_cell(ci, cj, ck);
        enters = in_md(md, S.nx, S.ny, cn);
        P.cell[p] = cn;
        P.ox[p] = o[0];
        P.oy[p] = o[1];
        P.oz[p] = o[2];
        deposit_global_fixed(rho, S, ci, cj, ck, o[0], o[1], o[2]);
      } else {
        P.cell[p] = -1;
      }
      P.vx[p] = v[0];
      P.vy[p] = v[1];
      P.vz[p] = v[2];
      t_w0 += st == ST_WALL0;
      t_w1 += st == ST_WALL1;
      t_bad += st == ST_BAD;
    }
    wave_append(enters, L.md_next, L.n_md_next, p);
  }
  outlier_tally(L, block0 * d->span, t_w0, t_w1, t_bad, t_coll, t_cap, t_fast);
}
__device__ __forceinline__ void outlier_block(const PIC_CONST PushDescF64* d, const PartF64& D, int do_mcc,
                                              int block0, int nblocks) {
  const PartF64 P = desc_records(d);
  const auto& S = d->S;
  const auto& L = d->L;
  const auto& md = d->md;
  const double2* __restrict__ E = d->E;
  double* __restrict__ rho = d->rho;
  const Segments sg = segments(L.out_cnt, L.tstart, block0, nblocks, d->span);
  if (sg.total == 0) return;
  int t_w0 = 0, t_w1 = 0, t_bad = 0, t_coll = 0, t_cap = 0, t_fast = 0;
  for (int base = 0; base < sg.total; base += 64) {
    const int idx = base + (int)threadIdx.x;
    bool enters = false;
    int p = segment_entry(sg, L.out, idx);
    if (idx < sg.total && p < 0) {
      p = ~p;
      enters = slot_alive(D, p) && in_md(md, S.nx, S.ny, slot_cell(D, p));
    } else if (idx < sg.total) {
      double x[3], v[3];
      load_d(P, p, x, v);
      const int i0 = (int)floor(x[0]), j0 = (int)floor(x[1]), k0 = (int)floor(x[2]);
      double Ep[3];
      gather_d(E, S, i0, j0, k0, x[0] - i0, x[1] - j0, x[2] - k0, Ep);
      const int st = push_one_f64(S, Ep, x, v);
      t_fast += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] >= S.vfast2;
      if (st == ST_ALIVE) {
        bool coll = false, capv = false;
        if (do_mcc) {
          const uint32_t id = P.id[p];
          const uint4 r = philox4x32_10(id, *S.step, kColl, (uint32_t)S.sp, S.key0, S.key1);
          if ((uint64_t)r.x < S.T_null) collide(S, id, v, coll, capv, p);
        }
        t_coll += coll;
        t_cap += capv;
        double part[8];
        const int c = store_d(P, p, x, v, S, part);
        enters = in_md(md, S.nx, S.ny, c);
        Tile none{};
        corner_add<double>(none, -1, nullptr, rho, S, cell_i(c), cell_j(c), cell_k(c), part);
      } else {
        kill(P, p);
        P.vx[p] = v[0];
        P.vy[p] = v[1];
        P.vz[p] = v[2];
      }
      t_w0 += st == ST_WALL0;
      t_w1 += st == ST_WALL1;
      t_bad += st == ST_BAD;
    }
    wave_append(enters, L.md_next, L.n_md_next, p);
  }
  outlier_tally(L, block0 * d->span, t_w0, t_w1, t_bad, t_coll, t_cap, t_fast);
}

// ---------------------------------------------------------------- collisions
// The collision candidates that found no room in the LDS of their push block,
// of `nblocks` push blocks from block0 (listed at the block's first tile).
template <typename PT, typename H, typename WL>
__device__ __forceinline__ void collide_block(const PT& P, const H& S, const WL& L, int block0,
                                              int nblocks, int span) {
  const Segments sg = segments(L.coll_cnt, L.tstart, block0, nblocks, span);
  if (sg.total == 0) return;
  int n_coll = 0, n_cap = 0;
  for (int base = 0; base < sg.total; base += 64) {
    const int idx = base + (int)threadIdx.x;
    const long p = segment_entry(sg, L.coll, idx);
    if (idx >= sg.total) continue;
    bool coll = false, capv = false;
    typename VelOf<PT>::type v[3] = {P.vx[p], P.vy[p], P.vz[p]};
    collide(S, P.id[p], v, coll, capv, p);
    if (coll) {
      P.vx[p] = v[0];
      P.vy[p] = v[1];
      P.vz[p] = v[2];
    }
    n_coll += coll;
    n_cap += capv;
  }
  n_coll = wave_sum(n_coll);
  n_cap = wave_sum(n_cap);
  if (threadIdx.x == 0) {
    unsigned long long* tl = L.tally + (long)TL_N * (block0 * span);
    tl[TL_COLL] += (unsigned long long)n_coll;
    tl[TL_CAP] += (unsigned long long)n_cap;
  }
}

// Everything after the push in one launch, one wave a block: nbmd blocks a
// species copy the MD particles' states back and collide them, `chunks` blocks
// to each push block near the MD cubes list the next step's, and the rest take
// the collision candidates and then the outliers of `group` push blocks each
// (disjoint sets of particles, one tally row).
template <typename PT, typename Desc>
__global__ __launch_bounds__(64) void lists_kernel(const Desc* descs, PT D0, PT D1, int npb,
                                                   int do_mcc, int nbmd, int near0, int near1,
                                                   int group, int chunks) {
  const PIC_CONST Desc* d = (const PIC_CONST Desc*)descs;
  int b = (int)blockIdx.x;
  if (b < 2 * nbmd) {
    const int sp = b >= nbmd ? 1 : 0;
    md_collide_block(d + sp, sp ? D1 : D0, b - sp * nbmd, nbmd, do_mcc);
    return;
  }
  b -= 2 * nbmd;
  if (b < near0 + near1) {
    const int sp = b >= near0 ? 1 : 0;
    near_block(d + sp, sp ? D1 : D0, b - sp * near0, chunks);
    return;
  }
  b -= near0 + near1;
  const int groups = (npb + group - 1) / group;
  const int sp = b >= groups ? 1 : 0;
  const int block0 = (b - sp * groups) * group, n = min(group, npb - block0);
  d += sp;
  if (do_mcc) collide_block(desc_records(d), d->S, d->L, block0, n, d->span);
  outlier_block(d, sp ? D1 : D0, do_mcc, block0, n);
}

// ---------------------------------------------------------------- loading
// Particle p of a species sits in cell p / ppc (x fastest); offsets are the top
// 24 bits of three Philox words (exact in FP32); velocities are Maxwellian by
// Box-Muller, per-component sigma = sqrt(kT/m), taken as v_{-1/2}.
__device__ __forceinline__ void load_draws(uint32_t p, int sp, uint32_t k0, uint32_t k1,
                                           double vth, double off[3], double vel[3]) {
  const uint4 a = philox4x32_10(p, 0u, kInitPos, (uint32_t)sp, k0, k1);
  off[0] = (double)(a.x >> 8) * 5.9604644775390625e-08;
  off[1] = (double)(a.y >> 8) * 5.9604644775390625e-08;
  off[2] = (double)(a.z >> 8) * 5.9604644775390625e-08;
  const uint4 b = philox4x32_10(p, 0u, kInitVel, (uint32_t)sp, k0, k1);
  double n0, n1, n2, n3;
  normal_pair(b.x, b.y, n0, n1);
  normal_pair(b.z, b.w, n2, n3);
  vel[0] = vth * n0;
  vel[1] = vth * n1;
  vel[2] = vth * n2;
}

__global__ void init_f64_kernel(PartF64 P, int n, int ppc, int nx, int ny, int sp, uint32_t k0,
                                uint32_t k1, double vth) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  const int cell = p / ppc;
  const int i = cell % nx, j = (cell / nx) % ny, k = cell / (nx * ny);
  double off[3], vel[3];
  load_draws((uint32_t)p, sp, k0, k1, vth, off, vel);
  P.x[p] = i + off[0];
  P.y[p] = j + off[1];
  P.z[p] = k + off[2];
  P.vx[p] = vel[0];
  P.vy[p] = vel[1];
  P.vz[p] = vel[2];
  P.id[p] = (uint32_t)p;
}

__global__ void init_f32r_kernel(PartF32R P, int n, int ppc, int nx, int ny, int sp, uint32_t k0,
                                 uint32_t k1, double vth) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  const int cell = p / ppc;
  double off[3], vel[3];
  load_draws((uint32_t)p, sp, k0, k1, vth, off, vel);
  P.cell[p] = pack_cell(cell % nx, (cell / nx) % ny, cell / (nx * ny));
  P.ox[p] = (float)off[0];
  P.oy[p] = (float)off[1];
  P.oz[p] = (float)off[2];
  P.vx[p] = (float)vel[0];
  P.vy[p] = (float)vel[1];
  P.vz[p] = (float)vel[2];
  P.id[p] = (uint32_t)p;
}

// ---------------------------------------------------------------- re-binning
// Counting sort of one species into the other buffer by tile, and by cell
// inside each tile, dropping the empty slots.  Each block takes kSortSlots
// consecutive slots of the (nearly binned) source:
//  1. count: the block's particles per destination tile, aggregated in an LDS
//     table, then one global atomic per (block, tile);
//  2. the tile sizes rounded up to a multiple of 4 and their exclusive scan
//     (the tile starts); each tile's cursor starts at its start; the padding
//     slots are marked empty;
//  3. scatter: per block again, one returning atomic per (block, tile)
//     reserves a contiguous run of the tile, and an LDS counting sort of the
//     block's particles by (tile, cell) places them in their runs in cell
//     order.
// A destination tile is thus a concatenation of cell-sorted runs, one per
// source block that sends particles into it (mostly one or two).  No atomic
// is taken per cell, so the cost does not grow with how far the particles
// have drifted since the last sort.
struct TileOrder {
  int ntx, nty;  // tiles along x, y
};
// key of a cell: tile index (tiles x fastest) * 64 + cell inside the tile (x fastest)
__device__ __forceinline__ int tiled_key(int i, int j, int k, TileOrder o) {
  return (((k >> 2) * o.nty + (j >> 2)) * o.ntx + (i >> 2)) * 64 + ((k & 3) * 4 + (j & 3)) * 4 +
         (i & 3);
}
__device__ __forceinline__ int sort_key(const PartF64& P, int p, TileOrder o) {
  if (!(P.z[p] >= 0.0)) return -1;
  return tiled_key((int)floor(P.x[p]), (int)floor(P.y[p]), (int)floor(P.z[p]), o);
}
__device__ __forceinline__ int sort_key(const PartF32R& P, int p, TileOrder o) {
  const int c = P.cell[p];
  if (c < 0) return -1;
  return tiled_key(cell_i(c), cell_j(c), cell_k(c), o);
}

// Runs of equal keys in neighbouring lanes (the input is nearly sorted): each
// lane learns the lane that heads its run, its rank in the run and, for the
// head, the run length, so one operation serves the whole run.
struct Run {
  int head, rank, len;
};
__device__ __forceinline__ Run lane_run(int key) {
  const int lane = threadIdx.x & 63;
  const int prev = __shfl_up(key, 1, 64);
  const bool is_head = lane == 0 || key != prev;
  const unsigned long long heads = __ballot(is_head);
  const unsigned long long upto = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
  Run r;
  r.head = 63 - __clzll((long long)(heads & upto));
  r.rank = lane - r.head;
  const unsigned long long above = lane == 63 ? 0ull : (heads & ~upto);
  r.len = (above ? __ffsll((long long)above) - 1 : 64) - lane;
  return r;
}

// Each wave takes kSortRounds rounds of 64 consecutive slots (a block covers
// kSortSlots slots); every load of a thread is issued before its first atomic.
constexpr int kSortRounds = 4;
constexpr int kSortSlots = 4 * 64 * kSortRounds;
constexpr int kTable = 64;  // destination tiles per block held in LDS (open addressing)

template <int Rounds = kSortRounds>
__device__ __forceinline__ int sort_first_slot() {
  return blockIdx.x * (256 * Rounds) + (threadIdx.x >> 6) * 64 * Rounds + (threadIdx.x & 63);
}
// rounds per wave of the scatter: half for FP64 records, so that a block's
// staged records fit in LDS
template <typename PT>
constexpr int scatter_rounds() {
  return std::is_same<PT, PartF64>::value ? kSortRounds / 2 : kSortRounds;
}

// the LDS table slot of tile t, inserted if new; -1 when the table is full
__device__ __forceinline__ int table_slot(int* s_tile, int t) {
  const unsigned h = ((unsigned)t * 2654435761u) >> 26;
  for (int probe = 0; probe < kTable; ++probe) {
    const int i = (int)((h + probe) & (kTable - 1));
    const int old = atomicCAS(&s_tile[i], -1, t);
    if (old == -1 || old == t) return i;
  }
  return -1;
}

template <typename PT>
__global__ __launch_bounds__(256) void bin_count_kernel(PT P, const int* __restrict__ cnt,
                                                        int* __restrict__ tcount, TileOrder o) {
  __shared__ int s_tile[kTable], s_n[kTable];
  if (threadIdx.x < kTable) {
    s_tile[threadIdx.x] = -1;
    s_n[threadIdx.x] = 0;
  }
  __syncthreads();
  const int n = cnt[0];
  const int first = sort_first_slot();
  int key[kSortRounds];
#pragma unroll
  for (int r = 0; r < kSortRounds; ++r) {
    const int p = first + 64 * r;
    key[r] = p < n ? sort_key(P, p, o) : -1;
  }
#pragma unroll
  for (int r = 0; r < kSortRounds; ++r) {
    const int t = key[r] >= 0 ? key[r] >> 6 : -1;
    const Run run = lane_run(t);
    if (t >= 0 && run.rank == 0) {
      const int sl = table_slot(s_tile, t);
      if (sl >= 0) atomicAdd(&s_n[sl], run.len);
      else atomicAdd(&tcount[t], run.len);
    }
  }
  __syncthreads();
  if (threadIdx.x < kTable && s_tile[threadIdx.x] >= 0)
    atomicAdd(&tcount[s_tile[threadIdx.x]], s_n[threadIdx.x]);
}

// one particle record in registers
struct RecF64 {
  double x, y, z, vx, vy, vz;
  uint32_t id;
};
struct RecF32R {
  int cell;
  float ox, oy, oz, vx, vy, vz;
  uint32_t id;
};
__device__ __forceinline__ void load_rec(const PartF64& a, int i, RecF64& r) {
  r.x = a.x[i];
  r.y = a.y[i];
  r.z = a.z[i];
  r.vx = a.vx[i];
  r.vy = a.vy[i];
  r.vz = a.vz[i];
  r.id = a.id[i];
}
__device__ __forceinline__ void store_rec(const PartF64& b, int j, const RecF64& r) {
  b.x[j] = r.x;
  b.y[j] = r.y;
  b.z[j] = r.z;
  b.vx[j] = r.vx;
  b.vy[j] = r.vy;
  b.vz[j] = r.vz;
  b.id[j] = r.id;
}
__device__ __forceinline__ int rec_key(const RecF64& r, TileOrder o) {
  if (!(r.z >= 0.0)) return -1;
  return tiled_key((int)floor(r.x), (int)floor(r.y), (int)floor(r.z), o);
}
__device__ __forceinline__ void load_rec(const PartF32R& a, int i, RecF32R& r) {
  r.cell = a.cell[i];
  r.ox = a.ox[i];
  r.oy = a.oy[i];
  r.oz = a.oz[i];
  r.vx = a.vx[i];
  r.vy = a.vy[i];
  r.vz = a.vz[i];
  r.id = a.id[i];
}
__device__ __forceinline__ void store_rec(const PartF32R& b, int j, const RecF32R& r) {
  b.cell[j] = r.cell;
  b.ox[j] = r.ox;
  b.oy[j] = r.oy;
  b.oz[j] = r.oz;
  b.vx[j] = r.vx;
  b.vy[j] = r.vy;
  b.vz[j] = r.vz;
  b.id[j] = r.id;
}
__device__ __forceinline__ int rec_key(const RecF32R& r, TileOrder o) {
  if (r.cell < 0) return -1;
  return tiled_key(cell_i(r.cell), cell_j(r.cell), cell_k(r.cell), o);
}
__device__ __forceinline__ int rec_cell(const RecF64& r) {
  return pack_cell((int)floor(r.x), (int)floor(r.y), (int)floor(r.z));
}
__device__ __forceinline__ int rec_cell(const RecF32R& r) { return r.cell; }
template <typename PT>
struct RecOf;
template <>
struct RecOf<PartF64> {
  using type = RecF64;
};
template <>
struct RecOf<PartF32R> {
  using type = RecF32R;
};

// LDS staging of a block's records (one array per field, so neighbouring
// lanes touch neighbouring words) and their destinations
template <typename Rec, int N>
struct SortStage;
template <int N>
struct SortStage<RecF32R, N> {
  int cell[N];
  float ox[N], oy[N], oz[N], vx[N], vy[N], vz[N];
  uint32_t id[N];
  int dest[N];
  __device__ void put(int u, const RecF32R& r) {
    cell[u] = r.cell;
    ox[u] = r.ox;
    oy[u] = r.oy;
    oz[u] = r.oz;
    vx[u] = r.vx;
    vy[u] = r.vy;
    vz[u] = r.vz;
    id[u] = r.id;
  }
  __device__ RecF32R get(int u) const {
    return RecF32R{cell[u], ox[u], oy[u], oz[u], vx[u], vy[u], vz[u], id[u]};
  }
};
template <int N>
struct SortStage<RecF64, N> {
  double x[N], y[N], z[N], vx[N], vy[N], vz[N];
  uint32_t id[N];
  int dest[N];
  __device__ void put(int u, const RecF64& r) {
    x[u] = r.x;
    y[u] = r.y;
    z[u] = r.z;
    vx[u] = r.vx;
    vy[u] = r.vy;
    vz[u] = r.vz;
    id[u] = r.id;
  }
  __device__ RecF64 get(int u) const {
    return RecF64{x[u], y[u], z[u], vx[u], vy[u], vz[u], id[u]};
  }
};

template <typename PT>
__global__ __launch_bounds__(256) void bin_scatter_kernel(PT src, PT dst, const int* __restrict__ cnt,
                                                          int* __restrict__ cursor, TileOrder o,
                                                          MdTables md, int nx, int ny,
                                                          int32_t* __restrict__ md_list,
                                                          int* __restrict__ n_md) {
  using Rec = typename RecOf<PT>::type;
  constexpr int kBins = kTable * 64;         // (table slot, cell in tile)
  constexpr int kPerThread = kBins / 256;    // bins scanned per thread
  __shared__ int s_tile[kTable], s_base[kTable];
  __shared__ int s_bin[kBins];
  __shared__ int s_wsum[4], s_mdbase;
  for (int i = threadIdx.x; i < kBins; i += 256) s_bin[i] = 0;
  if (threadIdx.x < kTable) s_tile[threadIdx.x] = -1;
  const int n = cnt[0];
  constexpr int R = scatter_rounds<PT>();
  const int first = sort_first_slot<R>();
  Rec rec[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int p = first + 64 * r;
    if (p < n) load_rec(src, p, rec[r]);
  }
  __syncthreads();
  int key[R], slot[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    key[r] = first + 64 * r < n ? rec_key(rec[r], o) : -1;
    const int t = key[r] >= 0 ? key[r] >> 6 : -1;
    const Run run = lane_run(t);
    int sl = -1;
    if (t >= 0 && run.rank == 0) sl = table_slot(s_tile, t);
    sl = __shfl(sl, run.head, 64);
    slot[r] = t >= 0 ? sl : -1;
    // one LDS atomic per run of equal bins (the input is nearly sorted)
    const int bk = slot[r] >= 0 ? slot[r] * 64 + (key[r] & 63) : -1;
    const Run brun = lane_run(bk);
    if (bk >= 0 && brun.rank == 0) atomicAdd(&s_bin[bk], brun.len);
  }
  __syncthreads();
  // exclusive scan of the bins in (slot, cell) order: block-local positions
  int local[kPerThread], sum = 0;
#pragma unroll
  for (int b = 0; b < kPerThread; ++b) {
    local[b] = s_bin[kPerThread * threadIdx.x + b];
    sum += local[b];
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int incl = sum;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int u = __shfl_up(incl, off, 64);
    if (lane >= off) incl += u;
  }
  if (lane == 63) s_wsum[w] = incl;
  __syncthreads();
  int run = incl - sum, total = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (k < w) run += s_wsum[k];
    total += s_wsum[k];
  }
#pragma unroll
  for (int b = 0; b < kPerThread; ++b) {
    s_bin[kPerThread * threadIdx.x + b] = run;
    run += local[b];
  }
  __syncthreads();
  // one reservation per (block, tile): the run of the tile this block fills
  if (threadIdx.x < kTable && s_tile[threadIdx.x] >= 0) {
    const int g0 = s_bin[64 * threadIdx.x];
    const int g1 = threadIdx.x + 1 < kTable ? s_bin[64 * (threadIdx.x + 1)] : total;
    s_base[threadIdx.x] = atomicAdd(&cursor[s_tile[threadIdx.x]], g1 - g0) - g0;
  }
  __syncthreads();
  // the records are staged in LDS at their block-local places and then
  // written out in destination order (whole lines)
  __shared__ SortStage<Rec, 256 * R> s_stage;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    // places in the bin: one LDS atomic per run, lanes of a run in lane order
    const int bk = slot[r] >= 0 ? slot[r] * 64 + (key[r] & 63) : -1;
    const Run brun = lane_run(bk);
    int d0 = 0;
    if (bk >= 0 && brun.rank == 0) d0 = atomicAdd(&s_bin[bk], brun.len);
    d0 = __shfl(d0, brun.head, 64);
    if (key[r] < 0) continue;
    if (slot[r] >= 0) {
      const int u = d0 + brun.rank;
      s_stage.put(u, rec[r]);
      s_stage.dest[u] = s_base[slot[r]] + u;
    } else {
      const int j = atomicAdd(&cursor[key[r] >> 6], 1);  // the table was full
      store_rec(dst, j, rec[r]);
      if (in_md(md, nx, ny, rec_cell(rec[r]))) md_list[atomicAdd(n_md, 1)] = j;
    }
  }
  __syncthreads();
  bool mine = false;  // any record of this thread that is in an MD cube
  for (int u = threadIdx.x; u < total; u += 256) {
    const Rec r = s_stage.get(u);
    store_rec(dst, s_stage.dest[u], r);
    if (md.n_grains > 0) mine = mine || in_md(md, nx, ny, rec_cell(r));
  }
  if (!__syncthreads_or(mine)) return;
  // those listed in destination order, one reservation per 256 (most blocks have none)
  for (int u0 = 0; u0 < total; u0 += 256) {
    const int u = u0 + (int)threadIdx.x;
    const bool in = u < total && in_md(md, nx, ny, rec_cell(s_stage.get(u)));
    const unsigned long long m = __ballot(in);
    __syncthreads();
    if (lane == 0) s_wsum[w] = __popcll(m);
    __syncthreads();
    if (threadIdx.x == 0) s_mdbase = atomicAdd(n_md, s_wsum[0] + s_wsum[1] + s_wsum[2] + s_wsum[3]);
    __syncthreads();
    int at = s_mdbase + __popcll(m & ((1ull << lane) - 1ull));
    for (int k = 0; k < w; ++k) at += s_wsum[k];
    if (in) md_list[at] = s_stage.dest[u];
  }
}

// t <= ngrid: the tile's size rounded up to a multiple of 4 (0 for the grid's
// padding tiles and the end entry), scanned afterwards into the tile starts
__global__ void tile_size_kernel(const int* __restrict__ tcount, int* __restrict__ tsize,
                                 int ngrid, int* __restrict__ n_md) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t == 0) *n_md = 0;  // the scatter lists the MD particles anew
  if (t > ngrid) return;
  tsize[t] = t < ngrid ? (tcount[t] + 3) & ~3 : 0;
}

// every tile's cursor at its start; its padding slots marked empty
template <typename PT>
__global__ void tile_pad_kernel(const int* __restrict__ tcount, const int* __restrict__ tstart,
                                int* __restrict__ cursor, PT dst, int ngrid) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= ngrid) return;
  const int s = tstart[t];
  cursor[t] = s;
  for (int p = s + tcount[t]; p < tstart[t + 1]; ++p) kill(dst, p);
}

// after the scatter the tiles fill [0, tstart[ngrid]) of the other buffer
__global__ void sort_finish_kernel(int* cnt, const int* tstart, int ngrid) {
  if (threadIdx.x == 0 && blockIdx.x == 0) cnt[0] = tstart[ngrid];
}

// exclusive scan of an int array: per-block sums, scan of the sums, per-block scan
constexpr int kScanBlock = 1024;
__global__ void scan_block_sums(const int* __restrict__ a, int n, int* __restrict__ sums) {
  __shared__ int s[kScanBlock];
  const int i = blockIdx.x * kScanBlock + threadIdx.x;
  s[threadIdx.x] = i < n ? a[i] : 0;
  __syncthreads();
  for (int off = kScanBlock / 2; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) s[threadIdx.x] += s[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) sums[blockIdx.x] = s[0];
}

__global__ void scan_sums_serial(int* __restrict__ sums, int nb, int* __restrict__ total) {
  __shared__ int s[kScanBlock];
  __shared__ int carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int base = 0; base < nb; base += kScanBlock) {
    const int i = base + threadIdx.x;
    const int v = i < nb ? sums[i] : 0;
    s[threadIdx.x] = v;
    __syncthreads();
    for (int off = 1; off < kScanBlock; off <<= 1) {
      const int t = (int)threadIdx.x >= off ? s[threadIdx.x - off] : 0;
      __syncthreads();
      s[threadIdx.x] += t;
      __syncthreads();
    }
    if (i < nb) sums[i] = carry + s[threadIdx.x] - v;
    __syncthreads();
    if (threadIdx.x == kScanBlock - 1) carry += s[threadIdx.x];
    __syncthreads();
  }
  if (threadIdx.x == 0 && total) *total = carry;
}

__global__ void scan_apply(const int* __restrict__ a, int n, const int* __restrict__ sums,
                           int* __restrict__ out) {
  __shared__ int s[kScanBlock];
  const int i = blockIdx.x * kScanBlock + threadIdx.x;
  const int v = i < n ? a[i] : 0;
  s[threadIdx.x] = v;
  __syncthreads();
  for (int off = 1; off < kScanBlock; off <<= 1) {
    const int t = (int)threadIdx.x >= off ? s[threadIdx.x - off] : 0;
    __syncthreads();
    s[threadIdx.x] += t;
    __syncthreads();
  }
  if (i < n) out[i] = sums[blockIdx.x] + s[threadIdx.x] - v;
}

__global__ void fill_int_kernel(int* a, long n, int v) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = v;
}

// ---------------------------------------------------------------- ionisation
// The ionisations of the step, after every particle has moved and collided
// and before any re-binning: in the order of the parent electrons' ids (an
// event's rank is the number of events with a smaller id), each makes an
// electron and an ion at the parent's new position, in the slots after the
// last tile's -- the range of the grid's last padding tile, whose push block
// takes them through the global-memory paths until the next re-binning puts
// them in their tiles -- with ids next_id[s] + rank.  The ejected electron
// takes the fraction s (Philox(id, k, IONIZE, 0) word 0) of the shared
// centre-of-mass energy, an isotropic direction (words 1 and 2), the neutral
// at rest; the ion a Maxwellian velocity of the gas temperature
// (Philox(id, k, IONIZE, 1), Box-Muller, cosine branch first).  Their charges
// cancel on the mesh (same position), so rho_{k+1} is left as it is.  If the
// new particles do not fit (room_* slots in use at most, so that the next
// re-binning fits too) or events exceeded the list, they are counted in
// *dropped.  One block.
constexpr int kIzThreads = 1024;
constexpr int kIzChunk = 4096;
__device__ __forceinline__ void copy_pos(const PartF64& s, long p, const PartF64& d, long q) {
  d.x[q] = s.x[p];
  d.y[q] = s.y[p];
  d.z[q] = s.z[p];
}
__device__ __forceinline__ void copy_pos(const PartF32R& s, long p, const PartF32R& d, long q) {
  d.cell[q] = s.cell[p];
  d.ox[q] = s.ox[p];
  d.oy[q] = s.oy[p];
  d.oz[q] = s.oz[p];
}

template <typename PT>
__global__ __launch_bounds__(kIzThreads) void ionize_kernel(PT Pe, PT Pi, WorkLists Le,
                                                            WorkLists Li, SpeciesStep Se,
                                                            MdTables md,
                                                            uint32_t* __restrict__ next_id,
                                                            long room_e, long room_i,
                                                            unsigned long long* dropped) {
  using V = typename VelOf<PT>::type;
  __shared__ uint32_t s_id[kIzChunk];
  const int total = *Se.iz_cnt;
  const int n = min(total, Se.iz_cap);
  const int ng = Le.ngrid;
  const long be = Le.tstart[ng], bi = Li.tstart[ng];
  // the tail stays a multiple of 4 slots long (a push thread streams four
  // slots at once): the slots after the new particles up to that are emptied
  const int n4 = (n + 3) & ~3;
  const bool fit = be + n4 <= room_e && bi + n4 <= room_i;
  const uint32_t k = *Se.step;
  for (int j0 = 0; fit && j0 < n; j0 += kIzThreads) {
    const int q = j0 + (int)threadIdx.x;
    const bool mine = q < n;
    const uint32_t myid = mine ? Se.iz_ev[q].id : 0u;
    int rank = 0;
    for (int c0 = 0; c0 < n; c0 += kIzChunk) {
      __syncthreads();
      for (int t = threadIdx.x; t < kIzChunk && c0 + t < n; t += kIzThreads) s_id[t] = Se.iz_ev[c0 + t].id;
      __syncthreads();
      const int m = min(kIzChunk, n - c0);
      if (mine)
        for (int t = 0; t < m; ++t) rank += s_id[t] < myid;
    }
    if (!mine) continue;
    const IzEvent ev = Se.iz_ev[q];
    const uint4 w0 = philox4x32_10(ev.id, k, kIonize, 0u, Se.key0, Se.key1);
    const uint4 w1 = philox4x32_10(ev.id, k, kIonize, 1u, Se.key0, Se.key1);
    const double ge = sqrt(u01_open(w0.x) * ev.gsq);
    const double cost = 1.0 - 2.0 * u01_open(w0.y);
    const double sint = sqrt(fmax(0.0, 1.0 - cost * cost));
    double sp, cp;
    sincos(2.0 * kPi * u01_open(w0.z), &sp, &cp);
    const double nh[3] = {sint * cp, sint * sp, cost};
    const long pe = be + rank, pi = bi + rank;
    copy_pos(Pe, ev.slot, Pe, pe);
    copy_pos(Pe, ev.slot, Pi, pi);
    Pe.vx[pe] = (V)(Se.mass_ratio_e * ev.v[0] + Se.mass_ratio_n * ge * nh[0]);
    Pe.vy[pe] = (V)(Se.mass_ratio_e * ev.v[1] + Se.mass_ratio_n * ge * nh[1]);
    Pe.vz[pe] = (V)(Se.mass_ratio_e * ev.v[2] + Se.mass_ratio_n * ge * nh[2]);
    double n0, n1, n2, n3;
    normal_pair(w1.x, w1.y, n0, n1);
    normal_pair(w1.z, w1.w, n2, n3);
    Pi.vx[pi] = (V)(Se.vth_gas * n0);
    Pi.vy[pi] = (V)(Se.vth_gas * n1);
    Pi.vz[pi] = (V)(Se.vth_gas * n2);
    Pe.id[pe] = next_id[0] + (uint32_t)rank;
    Pi.id[pi] = next_id[1] + (uint32_t)rank;
    if (in_md(md, Se.nx, Se.ny, slot_cell(Pe, ev.slot))) {
      Le.md_next[atomicAdd(Le.n_md_next, 1)] = (int32_t)pe;
      Li.md_next[atomicAdd(Li.n_md_next, 1)] = (int32_t)pi;
    }
  }
  if (fit && (int)threadIdx.x < n4 - n) {
    kill(Pe, be + n + threadIdx.x);
    kill(Pi, bi + n + threadIdx.x);
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  if (fit && n > 0) {
    Le.tstart[ng] = (int32_t)(be + n4);
    Li.tstart[ng] = (int32_t)(bi + n4);
    Le.cnt[0] = (int32_t)(be + n4);
    Li.cnt[0] = (int32_t)(bi + n4);
    next_id[0] += (uint32_t)n;
    next_id[1] += (uint32_t)n;
    Le.tally[TL_BORN] += (unsigned long long)n;
    Li.tally[TL_BORN] += (unsigned long long)n;
  }
  const int lost = fit ? total - n : total;
  if (lost > 0) *dropped += (unsigned long long)lost;
  *Se.iz_cnt = 0;
}

// ---------------------------------------------------------------- energy
// FP64 energy diagnostic.  Per block: the sum of |v|^2 over the live slots it
// strides (kinetic), or of |E|^2 times the node's share of a cell volume (half
// on the two electrode planes) over the nodes it strides (field); block b
// writes out[b].  A fixed grid and order make the sums repeatable.
constexpr int kEnergyBlocks = 1024;
__device__ __forceinline__ double block_sum(double v) {
  __shared__ double s_w[kBlock / 64];
  v = wave_sum_t<double>(v);
  if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < kBlock / 64; ++w) t += s_w[w];
  return t;
}

template <typename PT>
__global__ __launch_bounds__(kBlock) void kinetic_kernel(PT P, const int32_t* __restrict__ cnt,
                                                         double* __restrict__ out) {
  const long slots = cnt[0];
  double s = 0.0;
  for (long p = (long)blockIdx.x * kBlock + threadIdx.x; p < slots; p += (long)gridDim.x * kBlock) {
    if (!slot_alive(P, p)) continue;
    const double vx = P.vx[p], vy = P.vy[p], vz = P.vz[p];
    s += vx * vx + vy * vy + vz * vz;
  }
  s = block_sum(s);
  if (threadIdx.x == 0) out[blockIdx.x] = s;
}

template <typename ET>
__global__ __launch_bounds__(kBlock) void field_energy_kernel(const ET* __restrict__ E, long nxy,
                                                              int nz, double* __restrict__ out) {
  const long nn = nxy * (nz + 1);
  double s = 0.0;
  for (long n = (long)blockIdx.x * kBlock + threadIdx.x; n < nn; n += (long)gridDim.x * kBlock) {
    double ex, ey, ez;
    load_node(E, n, ex, ey, ez);
    const long k = n / nxy;
    s += (k == 0 || k == nz ? 0.5 : 1.0) * (ex * ex + ey * ey + ez * ez);
  }
  s = block_sum(s);
  if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// ---------------------------------------------------------------- launchers
static inline int nblk(long n, int b) { return (int)((n + b - 1) / b); }

int tile_grid(int nx, int ny, int nz, int extra) {
  return (((nx + 3) / 4) * ((ny + 3) / 4) * ((nz + 3) / 4) + extra + 15) / 16 * 16;
}

void launch_push(const PushDescF64* descs, const WorkLists& L, bool move, hipStream_t st) {
  if (L.ngrid <= 0) return;
  const int span = push_span(L), nb = L.ngrid / span, chunk = push_chunk(L, span);
  if (move)
    hipLaunchKernelGGL(push_f64_kernel<true>, dim3(2 * nb), dim3(kBlock), 0, st, descs, nb, span, chunk);
  else
    hipLaunchKernelGGL(push_f64_kernel<false>, dim3(2 * nb), dim3(kBlock), 0, st, descs, nb, span, chunk);
}
void launch_push(const PushDescF32* descs, const WorkLists& L, bool move, hipStream_t st) {
  if (L.ngrid <= 0) return;
  const int span = push_span(L), nb = L.ngrid / span, chunk = push_chunk(L, span);
  if (move)
    hipLaunchKernelGGL(push_f32r_kernel<true>, dim3(2 * nb), dim3(kBlock), 0, st, descs, nb, span, chunk);
  else
    hipLaunchKernelGGL(push_f32r_kernel<false>, dim3(2 * nb), dim3(kBlock), 0, st, descs, nb, span, chunk);
}

void launch_push_batch_f32r(const PushDescF32* descs, const int32_t* start, int ndesc, int items,
                            hipStream_t st) {
  if (ndesc <= 0 || items <= 0) return;
  hipLaunchKernelGGL(push_batch_f32r_kernel, dim3(items), dim3(kBlock), 0, st, descs, start, ndesc);
}

constexpr int kMdBlocks = kMdTallyRows;

void launch_field_out(const double* psi, double* phi, void* E, int e_f64,
                      unsigned long long* zero_next, const double* b, double* partials,
                      const MdTables& md, const WorkLists L[2], int nx, int ny, int nz, double dx,
                      RfDrive rf, hipStream_t st) {
  const int planes = field_out_planes(nx * ny, nz), nbe = (int)field_out_sums(nx * ny, nz);
  const int nbm = md.n_grains > 0 ? nblk(8L * md.bsx * md.bsy * md.bsz, 256) : 0;
  if (e_f64)
    hipLaunchKernelGGL(field_out_kernel<double2>, dim3(nbe + nbm), dim3(256), 0, st, psi, phi,
                       (double2*)E, zero_next, b, partials, md, L[0].n_md_next, L[1].n_md_next, nx, ny,
                       nz, dx, rf, nbm, planes);
  else
    hipLaunchKernelGGL(field_out_kernel<float4>, dim3(nbe + nbm), dim3(256), 0, st, psi, phi,
                       (float4*)E, zero_next, b, partials, md, L[0].n_md_next, L[1].n_md_next, nx, ny,
                       nz, dx, rf, nbm, planes);
}

// waves for the particles that the loading density puts into the cubes, per
// species (the kernel strides over what there is)
static long md_particles(const MdTables& md, const SpeciesStep& S, const WorkLists& L) {
  return (long)(md.n_cells * (L.slots / ((double)S.nx * S.ny * S.nz)));
}
static int md_waves(const MdTables& md, const SpeciesStep& S, const WorkLists& L) {
  const long guess = md_particles(md, S, L), per = guess <= kMdQuad ? 16 : 64;
  return (int)std::min<long>(kMdBlocks, std::max<long>(64, guess / per * 5 / 4));
}
template <typename PT, typename ET, typename RT>
static void md_move_impl(const PT P[2], const PT D[2], const void* E, void* rho, const MdTables& md,
                         const SpeciesStep S[2], unsigned long long* gc, const WorkLists L[2],
                         hipStream_t st) {
  if (md.n_grains == 0 || L[0].ngrid <= 0) return;
  const int nb = md_waves(md, S[0], L[0]);
  SpeciesPair<PT> pr{{P[0], P[1]}, {S[0], S[1]}, {L[0], L[1]}, nb};
  hipLaunchKernelGGL((md_kernel<PT, ET, RT>), dim3(2 * nb), dim3(kMdThreads), 0, st, pr,
                     D[0], D[1], (const ET*)E, (RT*)rho, md, gc);
}
void launch_md_move(const PartF64 P[2], const PartF64 D[2], const void* E, void* rho,
                    const MdTables& md, const SpeciesStep S[2], unsigned long long* gc,
                    const WorkLists L[2], hipStream_t st) {
  md_move_impl<PartF64, double2, double>(P, D, E, rho, md, S, gc, L, st);
}
void launch_md_move(const PartF32R P[2], const PartF32R D[2], const void* E, void* rho,
                    const MdTables& md, const SpeciesStep S[2], unsigned long long* gc,
                    const WorkLists L[2], hipStream_t st) {
  md_move_impl<PartF32R, float4, long long>(P, D, E, rho, md, S, gc, L, st);
}

// two blocks a CU
constexpr int kResident = 512;
bool push_md_fits(const MdTables& md, const SpeciesStep& S, const WorkLists& L) {
  return md.n_grains > 0 && L.ngrid > 0 && md_particles(md, S, L) <= kMdQuad &&
         2 * (L.ngrid / push_span(L) + (md_waves(md, S, L) + 3) / 4) <= kResident;
}
template <typename PT, typename Desc, typename ET, typename RT>
static void push_md_impl(const Desc* descs, const PT P[2], const PT D[2], const void* E, void* rho,
                         const MdTables& md, const SpeciesStep S[2], unsigned long long* gc,
                         const WorkLists L[2], hipStream_t st) {
  const int span = push_span(L[0]), nb = L[0].ngrid / span;
  const int nm = (md_waves(md, S[0], L[0]) + 3) / 4;
  SpeciesPair<PT> pr{{P[0], P[1]}, {S[0], S[1]}, {L[0], L[1]}, nm};
  hipLaunchKernelGGL((push_md_kernel<PT, Desc, ET, RT>), dim3(2 * (nm + nb)), dim3(kBlock), 0, st,
                     descs, nb, span, push_chunk(L[0], span), pr, D[0], D[1], (const ET*)E, (RT*)rho,
                     md, gc);
}
void launch_push_md(const PushDescF64* descs, const PartF64 P[2], const PartF64 D[2], const void* E,
                    void* rho, const MdTables& md, const SpeciesStep S[2], unsigned long long* gc,
                    const WorkLists L[2], hipStream_t st) {
  push_md_impl<PartF64, PushDescF64, double2, double>(descs, P, D, E, rho, md, S, gc, L, st);
}
void launch_push_md(const PushDescF32* descs, const PartF32R P[2], const PartF32R D[2],
                    const void* E, void* rho, const MdTables& md, const SpeciesStep S[2],
                    unsigned long long* gc, const WorkLists L[2], hipStream_t st) {
  push_md_impl<PartF32R, PushDescF32, float4, long long>(descs, P, D, E, rho, md, S, gc, L, st);
}

std::vector<int32_t> near_blocks(const WorkLists& L, const MdTables& md, int nx, int ny, int nz,
                                 int margin, bool f64) {
  std::vector<int32_t> v;
  const int span = push_span(L);
  for (int t = 0; md.n_grains > 0 && t < L.ngrid; t += span)
    if (window_meets_md(make_tile(t, L, nx, ny, nz, margin, f64 ? kWinF64 : kWinF32, span), md, nx, ny))
      v.push_back(t);
  return v;
}

bool same_windows(const WorkLists& L, int nx, int ny, int nz, int m0, int m1, bool f64) {
  const int span = push_span(L), cap = f64 ? kWinF64 : kWinF32;
  for (int t = 0; t < L.ngrid; t += span) {
    const Tile a = make_tile(t, L, nx, ny, nz, m0, cap, span), b = make_tile(t, L, nx, ny, nz, m1, cap, span);
    if (a.x0 != b.x0 || a.y0 != b.y0 || a.k0 != b.k0 || a.tx != b.tx || a.ty != b.ty || a.tz != b.tz) return false;
  }
  return true;
}

constexpr int kMdListBlocks = 512;  // per species (tally rows 0 .. 511 of the MD rows)
template <typename PT, typename Desc>
static void lists_impl(const Desc* descs, const PT D[2], bool grains, const WorkLists L[2],
                       int do_mcc, hipStream_t st) {
  if (L[0].ngrid <= 0) return;
  const int npb = L[0].ngrid / push_span(L[0]), nbmd = grains ? kMdListBlocks : 0;
  // waves per near push block: its slots if the particles were spread evenly
  const long slots = L[0].slots / std::max(1, npb);
  const int chunks = (int)std::min<long>(64, std::max<long>(1, (slots + kNearSlots - 1) / kNearSlots));
  // push blocks per wave: about 4,096 waves a species (more than the chip holds
  // at once), so a wave has some entries to pack
  const int group = std::min(64, std::max(1, npb / 4096)), groups = (npb + group - 1) / group;
  const int n0 = L[0].n_near * chunks, n1 = L[1].n_near * chunks;
  hipLaunchKernelGGL((lists_kernel<PT, Desc>), dim3(2 * nbmd + n0 + n1 + 2 * groups), dim3(64), 0, st,
                     descs, D[0], D[1], npb, do_mcc, nbmd, n0, n1, group, chunks);
}
void launch_lists(const PushDescF64* descs, const PartF64 D[2], bool grains, const WorkLists L[2],
                  int do_mcc, hipStream_t st) {
  lists_impl(descs, D, grains, L, do_mcc, st);
}
void launch_lists(const PushDescF32* descs, const PartF32R D[2], bool grains, const WorkLists L[2],
                  int do_mcc, hipStream_t st) {
  lists_impl(descs, D, grains, L, do_mcc, st);
}

void launch_init_f64(const PartF64& P, int n, int ppc, int nx, int ny, int sp, uint32_t k0,
                     uint32_t k1, double vth, hipStream_t st) {
  if (n <= 0) return;
  hipLaunchKernelGGL(init_f64_kernel, dim3(nblk(n, 256)), dim3(256), 0, st, P, n, ppc, nx, ny, sp,
                     k0, k1, vth);
}

void launch_init_f32r(const PartF32R& P, int n, int ppc, int nx, int ny, int sp, uint32_t k0,
                      uint32_t k1, double vth, hipStream_t st) {
  if (n <= 0) return;
  hipLaunchKernelGGL(init_f32r_kernel, dim3(nblk(n, 256)), dim3(256), 0, st, P, n, ppc, nx, ny, sp,
                     k0, k1, vth);
}

template <int kT, int kCap, typename PT>
static void moments_launch(const PT& P, const SpeciesStep& S, const WorkLists& L, double* mom,
                           long nn, const AvgBins& avg, int nodes, hipStream_t st) {
  const long layer = (long)L.ntx * L.nty, pad = L.ngrid - layer * L.ntz;
  const dim3 grid(L.ntx, L.nty, L.ntz + (unsigned)((pad + layer - 1) / layer));
  using V = typename VelOf<PT>::type;
  hipLaunchKernelGGL((moments_kernel<PT, kT, kCap>), grid, dim3(kT),
                     mom_lds(nodes, kCap, sizeof(V)), st, P, S, L, mom, nn, avg, nodes);
}

int moments_setup() {
  const void* k[] = {(const void*)moments_kernel<PartF64, 512, kMomCapHalf>,
                     (const void*)moments_kernel<PartF32R, 512, kMomCapFull>,
                     (const void*)moments_kernel<PartF32R, 512, kMomCapHalf>,
                     (const void*)moments_kernel<PartF32R, 256, kMomCapHalf>};
  const int most = (int)mom_lds(kMomWin, kMomCapFull, sizeof(float));
  for (const void* f : k)
    if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, most) != hipSuccess) return -1;
  return 0;
}

void launch_moments(const PartF64* P64, const PartF32R* P32, const SpeciesStep& S,
                    const WorkLists& L, double* mom, long nn, const AvgBins& avg,
                    hipStream_t st) {
  if (L.ngrid <= 0) return;
  // the largest window: 4 cells and the margin on both sides along each axis
  const int m = std::min(S.margin, 2), edge = 5 + 2 * m, nodes = edge * edge * edge;
  if (P64)
    moments_launch<512, kMomCapHalf>(*P64, S, L, mom, nn, avg, nodes, st);
  else if (L.slots / L.ngrid > kMomCapHalf * 3 / 2)  // (slots with their headroom)
    moments_launch<512, kMomCapFull>(*P32, S, L, mom, nn, avg, nodes, st);
  else if (m > 1)
    moments_launch<512, kMomCapHalf>(*P32, S, L, mom, nn, avg, nodes, st);
  else
    moments_launch<256, kMomCapHalf>(*P32, S, L, mom, nn, avg, nodes, st);
}

template <typename PT>
static void fine_moments_impl(const PT P[2], const WorkLists L[2], const FineBox& fb, double* mom,
                              const AvgBins& avg, long capacity, hipStream_t st) {
  const int blocks = (int)std::min<long>(nblk(capacity, 256), 4096);
  if (blocks <= 0) return;
  hipLaunchKernelGGL(fine_moments_kernel<PT>, dim3(blocks, 2), dim3(256), 0, st, P[0], P[1],
                     L[0].tstart + L[0].ngrid, L[1].tstart + L[1].ngrid, fb, mom, avg);
}
void launch_fine_moments(const PartF64 P[2], const WorkLists L[2], const FineBox& fb, double* mom,
                         const AvgBins& avg, long capacity, hipStream_t st) {
  fine_moments_impl(P, L, fb, mom, avg, capacity, st);
}
void launch_fine_moments(const PartF32R P[2], const WorkLists L[2], const FineBox& fb, double* mom,
                         const AvgBins& avg, long capacity, hipStream_t st) {
  fine_moments_impl(P, L, fb, mom, avg, capacity, st);
}

void launch_ionize(const PartF64* Pe64, const PartF64* Pi64, const PartF32R* Pe32,
                   const PartF32R* Pi32, const WorkLists& Le, const WorkLists& Li,
                   const SpeciesStep& Se, const MdTables& md, uint32_t* next_id, long room_e,
                   long room_i, unsigned long long* dropped, hipStream_t st) {
  if (Pe64)
    hipLaunchKernelGGL(ionize_kernel<PartF64>, dim3(1), dim3(kIzThreads), 0, st, *Pe64, *Pi64, Le,
                       Li, Se, md, next_id, room_e, room_i, dropped);
  else
    hipLaunchKernelGGL(ionize_kernel<PartF32R>, dim3(1), dim3(kIzThreads), 0, st, *Pe32, *Pi32, Le,
                       Li, Se, md, next_id, room_e, room_i, dropped);
}

int energy_blocks() { return kEnergyBlocks; }

void launch_energy(const PartF64* P64, const PartF32R* P32, const WorkLists& L, double* out,
                   hipStream_t st) {
  if (P64)
    hipLaunchKernelGGL(kinetic_kernel<PartF64>, dim3(kEnergyBlocks), dim3(kBlock), 0, st, *P64,
                       L.cnt, out);
  else
    hipLaunchKernelGGL(kinetic_kernel<PartF32R>, dim3(kEnergyBlocks), dim3(kBlock), 0, st, *P32,
                       L.cnt, out);
}

void launch_field_energy(const void* E, int e_f64, long nxy, int nz, double* out, hipStream_t st) {
  if (e_f64)
    hipLaunchKernelGGL(field_energy_kernel<double2>, dim3(kEnergyBlocks), dim3(kBlock), 0, st,
                       (const double2*)E, nxy, nz, out);
  else
    hipLaunchKernelGGL(field_energy_kernel<float4>, dim3(kEnergyBlocks), dim3(kBlock), 0, st,
                       (const float4*)E, nxy, nz, out);
}

void launch_fill_int(int* a, long n, int v, hipStream_t st) {
  if (n <= 0) return;
  hipLaunchKernelGGL(fill_int_kernel, dim3(nblk(n, 256)), dim3(256), 0, st, a, n, v);
}

long sort_keys(int ngrid) { return 2L * ngrid + 1; }

template <typename PT>
static void sort_impl(const PT& src, const PT& dst, const WorkLists& L, const MdTables& md, int nx,
                      int ny, int32_t* md_list, int* n_md, int* hist, int* sums, long capacity,
                      hipStream_t st) {
  const TileOrder o{L.ntx, L.nty};
  const int ng = L.ngrid;
  int* tcount = hist;            // [ngrid + 1]
  int* cursor = hist + ng + 1;   // [ngrid]
  launch_fill_int(hist, 2L * ng + 1, 0, st);
  hipLaunchKernelGGL(bin_count_kernel<PT>, dim3(nblk(capacity, kSortSlots)), dim3(256), 0, st, src,
                     L.cnt, tcount, o);
  const int n = ng + 1;
  hipLaunchKernelGGL(tile_size_kernel, dim3(nblk(n, 256)), dim3(256), 0, st, tcount, L.tstart, ng,
                     n_md);
  const int nb = nblk(n, kScanBlock);
  hipLaunchKernelGGL(scan_block_sums, dim3(nb), dim3(kScanBlock), 0, st, L.tstart, n, sums);
  hipLaunchKernelGGL(scan_sums_serial, dim3(1), dim3(kScanBlock), 0, st, sums, nb, L.cnt + 4);
  hipLaunchKernelGGL(scan_apply, dim3(nb), dim3(kScanBlock), 0, st, L.tstart, n, sums, L.tstart);
  hipLaunchKernelGGL(tile_pad_kernel<PT>, dim3(nblk(ng, 256)), dim3(256), 0, st, tcount, L.tstart,
                     cursor, dst, ng);
  hipLaunchKernelGGL(bin_scatter_kernel<PT>, dim3(nblk(capacity, 256 * scatter_rounds<PT>())),
                     dim3(256), 0, st,
                     src, dst, L.cnt, cursor, o, md, nx, ny, md_list, n_md);
  hipLaunchKernelGGL(sort_finish_kernel, dim3(1), dim3(64), 0, st, L.cnt, L.tstart, ng);
}

void launch_sort(const PartF64& src, const PartF64& dst, const WorkLists& L, const MdTables& md,
                 int nx, int ny, int32_t* md_list, int* n_md, int* hist, int* sums, long capacity,
                 hipStream_t st) {
  if (capacity > 0) sort_impl(src, dst, L, md, nx, ny, md_list, n_md, hist, sums, capacity, st);
}
void launch_sort(const PartF32R& src, const PartF32R& dst, const WorkLists& L, const MdTables& md,
                 int nx, int ny, int32_t* md_list, int* n_md, int* hist, int* sums, long capacity,
                 hipStream_t st) {
  if (capacity > 0) sort_impl(src, dst, L, md, nx, ny, md_list, n_md, hist, sums, capacity, st);
}

}  // namespace pic
