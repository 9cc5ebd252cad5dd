// spectral.hip -- the Poisson solve of Eq. (3) in FP64 on the half spectrum
// (gfx950): real FFTs along the periodic x, y and tridiagonal solves along z.
//
// The charge is real, so of the nx Fourier columns only hx = nx / 2 + 1 are
// independent.  Two real rows y = 2 j, 2 j + 1 are transformed as one complex
// row (one as the real, the other as the imaginary part) and separated after
// it; the y lines, the tridiagonal solves and the work array then hold hx
// columns: FP64 costs the bytes and the line count that a full complex FP32
// transform would.  Everything here is bound by latency (a plane's few
// butterflies per thread, the barriers between the stages) up to 64x64 planes
// and by the work array's traffic beyond.
//
// Measured against the transforms of the full spectrum that this replaces
// (FP64: line transforms through HBM with separate right-hand-side, grain and
// electrode kernels; FP32R: two FP32 sweeps with their residuals and norms),
// whole field stage with the field kernel: 64x64x256 FP64 104 -> 58 us, FP32R
// 148 -> 60 us; 16x16x32 FP64 33 -> 22 us in 4 launches for 7, FP32R 62 ->
// 23 us in 4 for 9; 128x128x512 FP32R 1,090 -> 390 us.  A block of 1,024 threads
// takes a 64x64 plane's rows forward in 17.2 us, one of 512 in 18.6, of 256 in
// 24.6 (FP32R); a 16x16 plane takes 8 us with any of them.
//
// kernels, in the order of a solve (K = nz - 1 interior planes):
//   rows_fwd   right-hand side, x rows; a whole plane per block with its y
//              lines too where two half-spectrum planes fit in LDS (plan.full),
//              else some row pairs per block
//   cols       y lines of the larger planes, in place, some columns per block
//   tridiag    every mode along z, in chunks
//   rows_inv   the inverse of rows_fwd
// The field kernel that follows reads psi's six neighbours anyway and forms
// the residual that the solve ended with (FP32R).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "device_common.hpp"
#include "launch.hpp"

namespace pic {

namespace {

__device__ __forceinline__ double2 c_add(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 c_sub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 c_scale(double2 a, double s) { return make_double2(a.x * s, a.y * s); }
// a w (forward: w conjugated; the tables hold exp(+2 pi i t / N))
template <bool kFwd>
__device__ __forceinline__ double2 c_tw(double2 a, double2 w) {
  const double wy = kFwd ? -w.y : w.y;
  return make_double2(a.x * w.x - a.y * wy, a.x * wy + a.y * w.x);
}
// a times -i (forward) or +i
template <bool kFwd>
__device__ __forceinline__ double2 c_rot(double2 a) {
  return kFwd ? make_double2(a.y, -a.x) : make_double2(-a.y, a.x);
}

template <bool kFwd>
__device__ __forceinline__ void dft3(double2 a0, double2 a1, double2 a2, double2* o) {
  constexpr double s3 = 0.86602540378443864676;
  const double2 t = c_add(a1, a2);
  const double2 u = make_double2(a0.x - 0.5 * t.x, a0.y - 0.5 * t.y);
  const double2 v = c_rot<kFwd>(c_scale(c_sub(a1, a2), s3));
  o[0] = c_add(a0, t);
  o[1] = c_add(u, v);
  o[2] = c_sub(u, v);
}
template <bool kFwd>
__device__ __forceinline__ void dft4(double2 a0, double2 a1, double2 a2, double2 a3, double2* o) {
  const double2 t0 = c_add(a0, a2), t1 = c_sub(a0, a2);
  const double2 t2 = c_add(a1, a3), t3 = c_rot<kFwd>(c_sub(a1, a3));
  o[0] = c_add(t0, t2);
  o[1] = c_add(t1, t3);
  o[2] = c_sub(t0, t2);
  o[3] = c_sub(t1, t3);
}
// the DFT of R values in registers
template <int R, bool kFwd>
__device__ __forceinline__ void dft(const double2* a, double2* o) {
  if constexpr (R == 2) {
    o[0] = c_add(a[0], a[1]);
    o[1] = c_sub(a[0], a[1]);
  } else if constexpr (R == 3) {
    dft3<kFwd>(a[0], a[1], a[2], o);
  } else if constexpr (R == 4) {
    dft4<kFwd>(a[0], a[1], a[2], a[3], o);
  } else if constexpr (R == 5) {
    // c_j + (-/+) i s_j with the cosines and sines of 2 pi / 5, 4 pi / 5
    constexpr double c1 = 0.30901699437494742410, c2 = -0.80901699437494742410;
    constexpr double s1 = 0.95105651629515357212, s2 = 0.58778525229247312917;
    const double2 p1 = c_add(a[1], a[4]), m1 = c_sub(a[1], a[4]);
    const double2 p2 = c_add(a[2], a[3]), m2 = c_sub(a[2], a[3]);
    const double2 u1 = make_double2(a[0].x + c1 * p1.x + c2 * p2.x, a[0].y + c1 * p1.y + c2 * p2.y);
    const double2 u2 = make_double2(a[0].x + c2 * p1.x + c1 * p2.x, a[0].y + c2 * p1.y + c1 * p2.y);
    const double2 v1 = c_rot<kFwd>(make_double2(s1 * m1.x + s2 * m2.x, s1 * m1.y + s2 * m2.y));
    const double2 v2 = c_rot<kFwd>(make_double2(s2 * m1.x - s1 * m2.x, s2 * m1.y - s1 * m2.y));
    o[0] = c_add(a[0], c_add(p1, p2));
    o[1] = c_add(u1, v1);
    o[2] = c_add(u2, v2);
    o[3] = c_sub(u2, v2);
    o[4] = c_sub(u1, v1);
  } else if constexpr (R == 6) {
    double2 e[3], q[3];
    dft3<kFwd>(a[0], a[2], a[4], e);
    dft3<kFwd>(a[1], a[3], a[5], q);
    constexpr double s3 = 0.86602540378443864676;
    q[1] = c_tw<kFwd>(q[1], make_double2(0.5, s3));
    q[2] = c_tw<kFwd>(q[2], make_double2(-0.5, s3));
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      o[j] = c_add(e[j], q[j]);
      o[j + 3] = c_sub(e[j], q[j]);
    }
  } else {  // 8
    double2 e[4], q[4];
    dft4<kFwd>(a[0], a[2], a[4], a[6], e);
    dft4<kFwd>(a[1], a[3], a[5], a[7], q);
    constexpr double h = 0.70710678118654752440;
    q[1] = c_scale(c_add(q[1], c_rot<kFwd>(q[1])), h);
    q[2] = c_rot<kFwd>(q[2]);
    q[3] = c_scale(c_sub(c_rot<kFwd>(q[3]), q[3]), h);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      o[j] = c_add(e[j], q[j]);
      o[j + 4] = c_sub(e[j], q[j]);
    }
  }
}

// b / d by the multiplier m = ceil(2^32 / d) (m = 0: d = 1); exact for
// b d < 2^32, and b stays below 2^20 here
__device__ __forceinline__ int div_by(int b, unsigned m) {
  return m ? (int)__umulhi((unsigned)b, m) : b;
}

// One Stockham stage of radix R over L lines of length N in LDS (decimation
// in frequency, s the product of the radices done, n = N / s, m = n / R):
//   y[q + s (R p + j)] = w_n^{j p} sum_k x[q + s (p + k m)] w_R^{j k}.
// Neighbouring lanes take neighbouring lines: with a line stride of 1, or an
// odd one for the rows, no two lanes of a group meet in a bank, and the
// twiddle is the same for the whole group.
template <int R, bool kFwd>
__device__ __forceinline__ void stage(const double2* __restrict__ src, double2* __restrict__ dst, int N, int L,
                                      unsigned mL, int ls, int es, int s, unsigned ms, int m,
                                      const double2* __restrict__ tw) {
  const int nb = L * (N / R);
  for (int b = (int)threadIdx.x; b < nb; b += (int)blockDim.x) {
    const int t = div_by(b, mL), l = b - t * L;
    const int p = div_by(t, ms), q = t - p * s;
    const double2* x = src + l * ls + t * es;  // q + s p = t
    double2* y = dst + l * ls + (q + s * R * p) * es;
    const int xs = s * m * es, ys = s * es;
    double2 a[R], o[R];
#pragma unroll
    for (int k = 0; k < R; ++k) a[k] = x[k * xs];
    dft<R, kFwd>(a, o);
    y[0] = o[0];
    if (m == 1) {  // the last stage: p = 0
#pragma unroll
      for (int j = 1; j < R; ++j) y[j * ys] = o[j];
    } else {
#pragma unroll
      for (int j = 1; j < R; ++j) y[j * ys] = c_tw<kFwd>(o[j], tw[j * p * s]);
    }
  }
  __syncthreads();
}

// every stage of L lines; returns the buffer that holds the result
template <bool kFwd>
__device__ double2* transform(double2* src, double2* dst, const FftLine& f, int L, unsigned mL, int ls, int es,
                              const double2* __restrict__ tw) {
  int s = 1, n = f.N;
  for (int i = 0; i < f.nst; ++i) {
    const int r = f.radix[i];
    const int m = n / r;
    const unsigned ms = f.mul_s[i];
    switch (r) {
      case 2: stage<2, kFwd>(src, dst, f.N, L, mL, ls, es, s, ms, m, tw); break;
      case 3: stage<3, kFwd>(src, dst, f.N, L, mL, ls, es, s, ms, m, tw); break;
      case 4: stage<4, kFwd>(src, dst, f.N, L, mL, ls, es, s, ms, m, tw); break;
      case 5: stage<5, kFwd>(src, dst, f.N, L, mL, ls, es, s, ms, m, tw); break;
      case 6: stage<6, kFwd>(src, dst, f.N, L, mL, ls, es, s, ms, m, tw); break;
      default: stage<8, kFwd>(src, dst, f.N, L, mL, ls, es, s, ms, m, tw); break;
    }
    double2* t = src;
    src = dst;
    dst = t;
    n = m;
    s *= r;
  }
  return src;
}

// the plasma's part of the right-hand side at interior node i
template <int kIn>
__device__ __forceinline__ double rhs_at(const SpectralArgs& a, long i, long plane) {
  if constexpr (kIn == kRhsRho64) return a.scale * a.rho64[i + plane];
  if constexpr (kIn == kRhsFixed) return a.scale * (double)a.rhofx[i + plane];
  return 0.0;
}
// one entry of the grains' shares of it
template <int kIn>
__device__ __forceinline__ double share_of(const SpectralArgs& a, const GrainShare& t) {
  if constexpr (kIn == kRhsUnit) return t.g == a.unit ? a.scale * t.w : 0.0;
  const long long net = (long long)a.counts[2 * t.g + 1] - (long long)a.counts[2 * t.g];
  if constexpr (kIn == kRhsFixed) return a.scale * (double)(net * t.part);
  return a.scale * (double)net * t.w;
}

// Right-hand side (FP32R: stored for the residual) and forward transform of the
// rows (and, whole planes, of the columns).  Block: `pairs` row pairs of one
// plane.  Block 0 freezes the grains' charges.
template <int kIn>
__global__ __launch_bounds__(kRowThreads) void rows_fwd_kernel(SpectralPlan pl, SpectralArgs a,
                                                               double2* __restrict__ work) {
  extern __shared__ unsigned char smem_raw[];
  const int nx = pl.fx.N, ny = pl.fy.N, hx = pl.hx, np = nx * ny;
  double2* tw_x = reinterpret_cast<double2*>(smem_raw);
  double2* tw_y = tw_x + nx;
  double2* b0 = tw_y + (pl.full ? ny : 0);
  double2* b1 = b0 + pl.buf;
  const int k = (int)blockIdx.x / pl.chunks, ch = (int)blockIdx.x - k * pl.chunks;
  const int j0 = ch * pl.pairs, nj = min(pl.pairs, pl.npair - j0);
  const long pbase = (long)k * np;
  const int e_beg = a.tab_start ? a.tab_start[blockIdx.x] : 0, e_end = a.tab_start ? a.tab_start[blockIdx.x + 1] : 0;
  if (kIn != kRhsUnit && blockIdx.x == 0)
    for (int q = (int)threadIdx.x; q < a.ng; q += (int)blockDim.x)
      a.Q[q] = (double)((long long)a.counts[2 * q + 1] - (long long)a.counts[2 * q]) * a.we;
  for (int t = (int)threadIdx.x; t < nx; t += (int)blockDim.x) tw_x[t] = a.tw_x[t];
  if (pl.full)
    for (int t = (int)threadIdx.x; t < ny; t += (int)blockDim.x) tw_y[t] = a.tw_y[t];
  __syncthreads();
  const int n_in = nj * nx;
#pragma unroll 4
  for (int u = (int)threadIdx.x; u < n_in; u += (int)blockDim.x) {
    const int jl = div_by(u, pl.mul_nx), x = u - jl * nx;
    const int y = 2 * (j0 + jl);
    const bool two = y + 1 < ny;
    const long i0 = pbase + (long)y * nx + x, i1 = two ? i0 + nx : i0;
    double2 v;
    v.x = rhs_at<kIn>(a, i0, np);
    v.y = two ? rhs_at<kIn>(a, i1, np) : 0.0;
    if constexpr (kIn == kRhsFixed) {
      a.b[i0] = v.x;
      if (two) a.b[i1] = v.y;
    }
    b0[jl * pl.ldx + x] = v;
  }
  __syncthreads();
  if (e_beg < e_end) {  // (block-uniform) the grains' shares: a thread per node that has any
    for (int e = e_beg + (int)threadIdx.x; e < e_end; e += (int)blockDim.x) {
      const int node = a.tab[e].node;
      if (e > e_beg && a.tab[e - 1].node == node) continue;
      double add = 0.0;
      for (int q = e; q < e_end && a.tab[q].node == node; ++q) add += share_of<kIn>(a, a.tab[q]);
      const int pn = (int)(node - pbase), y = pn / nx, x = pn - y * nx;
      double2& v = b0[(y / 2 - j0) * pl.ldx + x];
      if (y & 1) v.y += add;
      else v.x += add;
      if (kIn == kRhsFixed) a.b[node] += add;
    }
    __syncthreads();
  }
  double2* z = transform<true>(b0, b1, pl.fx, nj, ch + 1 == pl.chunks ? pl.mul_last : pl.mul_pairs, pl.ldx, 1, tw_x);
  double2* h = z == b0 ? b1 : b0;
  // the two rows of a pair: A = (Z_m + conj Z_-m) / 2, B = (Z_m - conj Z_-m) / 2i
  const int n_sp = nj * hx;
  double2* out = work + ((long)k * ny + 2 * j0) * hx;
  for (int u = (int)threadIdx.x; u < n_sp; u += (int)blockDim.x) {
    const int jl = div_by(u, pl.mul_hx), m = u - jl * hx;
    const double2 p = z[jl * pl.ldx + m], q = z[jl * pl.ldx + (m ? nx - m : 0)];
    const double2 A = make_double2(0.5 * (p.x + q.x), 0.5 * (p.y - q.y));
    const double2 B = make_double2(0.5 * (p.y + q.y), 0.5 * (q.x - p.x));
    double2* o = pl.full ? h : out;
    o[(2 * jl) * hx + m] = A;
    if (2 * (j0 + jl) + 1 < ny) o[(2 * jl + 1) * hx + m] = B;
  }
  if (!pl.full) return;
  __syncthreads();
  const double2* res = transform<true>(h, z, pl.fy, hx, pl.mul_hx, 1, hx, tw_y);
  for (int u = (int)threadIdx.x; u < ny * hx; u += (int)blockDim.x) out[u] = res[u];
}

// The inverse: (whole planes: columns, then) rows, and the real values times
// 1 / (nx ny) stored as psi.
__global__ __launch_bounds__(kRowThreads) void rows_inv_kernel(SpectralPlan pl, const double2* __restrict__ gtw_x,
                                                               const double2* __restrict__ gtw_y,
                                                               const double2* __restrict__ work,
                                                               double* __restrict__ psi) {
  extern __shared__ unsigned char smem_raw[];
  const int nx = pl.fx.N, ny = pl.fy.N, hx = pl.hx, np = nx * ny;
  double2* tw_x = reinterpret_cast<double2*>(smem_raw);
  double2* tw_y = tw_x + nx;
  double2* b0 = tw_y + (pl.full ? ny : 0);
  double2* b1 = b0 + pl.buf;
  const int k = (int)blockIdx.x / pl.chunks, ch = (int)blockIdx.x - k * pl.chunks;
  const int j0 = ch * pl.pairs, nj = min(pl.pairs, pl.npair - j0);
  const int rows = min(ny, 2 * (j0 + nj)) - 2 * j0;
  const double2* in = work + ((long)k * ny + 2 * j0) * hx;
  for (int u = (int)threadIdx.x; u < rows * hx; u += (int)blockDim.x) b0[u] = in[u];
  for (int t = (int)threadIdx.x; t < nx; t += (int)blockDim.x) tw_x[t] = gtw_x[t];
  if (pl.full)
    for (int t = (int)threadIdx.x; t < ny; t += (int)blockDim.x) tw_y[t] = gtw_y[t];
  __syncthreads();
  double2* h = b0;
  if (pl.full) h = transform<false>(b0, b1, pl.fy, hx, pl.mul_hx, 1, hx, tw_y);
  double2* z = h == b0 ? b1 : b0;
  // Z = A + i B on the first half, conj A + i conj B on the second
  for (int u = (int)threadIdx.x; u < nj * nx; u += (int)blockDim.x) {
    const int jl = div_by(u, pl.mul_nx), x = u - jl * nx;
    const bool low = x < hx;
    const int m = low ? x : nx - x;
    double2 A = h[2 * jl * hx + m];
    double2 B = 2 * jl + 1 < rows ? h[(2 * jl + 1) * hx + m] : make_double2(0.0, 0.0);
    if (!low) {
      A.y = -A.y;
      B.y = -B.y;
    }
    z[jl * pl.ldx + x] = make_double2(A.x - B.y, A.y + B.x);
  }
  __syncthreads();
  const double2* res = transform<false>(z, h, pl.fx, nj, ch + 1 == pl.chunks ? pl.mul_last : pl.mul_pairs, pl.ldx, 1, tw_x);
  const double s = 1.0 / (double)np;
  double* out = psi + (long)k * np + (long)2 * j0 * nx;
  for (int u = (int)threadIdx.x; u < nj * nx; u += (int)blockDim.x) {
    const int jl = div_by(u, pl.mul_nx), x = u - jl * nx;
    const double2 v = res[jl * pl.ldx + x];
    double* o = out + (long)2 * jl * nx + x;
    o[0] = v.x * s;
    if (2 * jl + 1 < rows) o[nx] = v.y * s;
  }
}

// the y lines of some columns of one plane, in place (planes too large for
// rows_fwd to take whole)
template <bool kFwd>
__global__ __launch_bounds__(256) void cols_kernel(SpectralPlan pl, const double2* __restrict__ gtw_y,
                                                   double2* __restrict__ work) {
  extern __shared__ unsigned char smem_raw[];
  const int ny = pl.fy.N, hx = pl.hx;
  double2* tw = reinterpret_cast<double2*>(smem_raw);
  double2* b0 = tw + ny;
  double2* b1 = b0 + pl.cols * ny;
  const int k = (int)blockIdx.x / pl.col_chunks, ch = (int)blockIdx.x - k * pl.col_chunks;
  const int m0 = ch * pl.cols, nc = min(pl.cols, hx - m0);
  const unsigned mul = ch + 1 == pl.col_chunks ? pl.mul_cols_last : pl.mul_cols;
  double2* g = work + (long)k * ny * hx + m0;
  for (int t = (int)threadIdx.x; t < ny; t += (int)blockDim.x) tw[t] = gtw_y[t];
#pragma unroll 4
  for (int u = (int)threadIdx.x; u < nc * ny; u += (int)blockDim.x) {
    const int y = div_by(u, mul), c = u - y * nc;
    b0[u] = g[(long)y * hx + c];
  }
  __syncthreads();
  const double2* res = transform<kFwd>(b0, b1, pl.fy, nc, mul, 1, nc, tw);
#pragma unroll 4
  for (int u = (int)threadIdx.x; u < nc * ny; u += (int)blockDim.x) {
    const int y = div_by(u, mul), c = u - y * nc;
    g[(long)y * hx + c] = res[u];
  }
}

// Tridiagonal solves along z: the two sweeps are first-order affine
// recurrences, forward y_k = f_k (d_k - y_{k-1}), backward
// x_k = y_k - f_k x_{k+1}, each split into kChunks chunks along z per mode.  A
// thread composes the affine map of its chunk (held in registers), the maps of
// the earlier chunks give its incoming value (LDS), and the chunk is re-run
// from it: the serial depth is K / kChunks + kChunks.  kModes modes a block:
// 128-byte rows and, at 33x64 modes, as many blocks as the chip has CUs.
// FP32R: one more block adds up the sums of the residual that the previous
// solve ended with and records its stopping test (see RefineState).
template <int kChunks, int kModes, int kLen>
__global__ __launch_bounds__(kChunks* kModes) void tridiag_kernel(double2* __restrict__ d,
                                                                  const double* __restrict__ inv, int K, long modes,
                                                                  RefineState rs) {
  __shared__ double s_A[kChunks][kModes];
  __shared__ double2 s_B[kChunks][kModes];
  if (rs.ctl && blockIdx.x + 1 == gridDim.x) {
    double rr = 0.0, bb = 0.0;
    for (int i = (int)threadIdx.x; i < rs.nb; i += kChunks * kModes) {
      rr += rs.partials[2 * (long)i];
      bb += rs.partials[2 * (long)i + 1];
    }
    double2* s = &s_B[0][0];
    s[threadIdx.x] = make_double2(rr, bb);
    __syncthreads();
    for (int off = kChunks * kModes / 2; off > 0; off >>= 1) {
      if ((int)threadIdx.x < off) s[threadIdx.x] = c_add(s[threadIdx.x], s[threadIdx.x + off]);
      __syncthreads();
    }
    if (threadIdx.x == 0) {
      if (rs.ctl[3]) {
        rs.norms[0] = s[0].x;
        rs.norms[1] = s[0].y;
        const int done = s[0].x <= rs.tol2 * s[0].y || s[0].x == 0.0;
        rs.ctl[0] = done;
        if (!done) rs.ctl[2] += 1;
      }
      rs.ctl[1] = 1;
      rs.ctl[3] = 1;
    }
    return;
  }
  const int lm = (int)threadIdx.x % kModes, c = (int)threadIdx.x / kModes;
  const long mn = (long)blockIdx.x * kModes + lm;
  const bool on = mn < modes;
  const int len = (K + kChunks - 1) / kChunks;
  const int k0 = c * len, n = on ? min(K - k0, len) : 0;
  double2 v[kLen];
  double f[kLen];
#pragma unroll
  for (int i = 0; i < kLen; ++i)
    if (i < n) {
      v[i] = d[(long)(k0 + i) * modes + mn];
      f[i] = inv[(long)(k0 + i) * modes + mn];
    }
  double A = 1.0;
  double2 B = make_double2(0.0, 0.0);
#pragma unroll
  for (int i = 0; i < kLen; ++i)
    if (i < n) {
      A = -f[i] * A;
      B.x = f[i] * (v[i].x - B.x);
      B.y = f[i] * (v[i].y - B.y);
    }
  s_A[c][lm] = A;
  s_B[c][lm] = B;
  __syncthreads();
  double2 y = make_double2(0.0, 0.0);
  for (int cc = 0; cc < c; ++cc) {
    const double a = s_A[cc][lm];
    const double2 b = s_B[cc][lm];
    y.x = a * y.x + b.x;
    y.y = a * y.y + b.y;
  }
#pragma unroll
  for (int i = 0; i < kLen; ++i)
    if (i < n) {
      y.x = f[i] * (v[i].x - y.x);
      y.y = f[i] * (v[i].y - y.y);
      v[i] = y;
    }
  __syncthreads();
  A = 1.0;
  B = make_double2(0.0, 0.0);
#pragma unroll
  for (int i = kLen - 1; i >= 0; --i)
    if (i < n) {
      A = -f[i] * A;
      B.x = v[i].x - f[i] * B.x;
      B.y = v[i].y - f[i] * B.y;
    }
  s_A[c][lm] = A;
  s_B[c][lm] = B;
  __syncthreads();
  double2 x = make_double2(0.0, 0.0);
  for (int cc = kChunks - 1; cc > c; --cc) {
    const double a = s_A[cc][lm];
    const double2 b = s_B[cc][lm];
    x.x = a * x.x + b.x;
    x.y = a * x.y + b.y;
  }
#pragma unroll
  for (int i = kLen - 1; i >= 0; --i)
    if (i < n) {
      x.x = v[i].x - f[i] * x.x;
      x.y = v[i].y - f[i] * x.y;
      d[(long)(k0 + i) * modes + mn] = x;
    }
}

// more than 32 x 32 planes: one thread per mode, the loads of a batch of
// planes issued together
__global__ __launch_bounds__(64) void tridiag_serial_kernel(double2* __restrict__ d, const double* __restrict__ inv,
                                                            int K, long modes) {
  constexpr int B = 8;
  const long mn = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (mn >= modes) return;
  double2 prev = make_double2(0.0, 0.0);
  for (int k0 = 0; k0 < K; k0 += B) {
    double2 cur[B];
    double f[B];
#pragma unroll
    for (int b = 0; b < B; ++b)
      if (k0 + b < K) {
        cur[b] = d[(long)(k0 + b) * modes + mn];
        f[b] = inv[(long)(k0 + b) * modes + mn];
      }
#pragma unroll
    for (int b = 0; b < B; ++b)
      if (k0 + b < K) {
        prev = make_double2((cur[b].x - prev.x) * f[b], (cur[b].y - prev.y) * f[b]);
        d[(long)(k0 + b) * modes + mn] = prev;
      }
  }
  double2 next = make_double2(0.0, 0.0);
  for (int k1 = K - 1; k1 >= 0; k1 -= B) {
    double2 cur[B];
    double f[B];
#pragma unroll
    for (int b = 0; b < B; ++b)
      if (k1 - b >= 0) {
        cur[b] = d[(long)(k1 - b) * modes + mn];
        f[b] = inv[(long)(k1 - b) * modes + mn];
      }
#pragma unroll
    for (int b = 0; b < B; ++b)
      if (k1 - b >= 0) {
        next = make_double2(cur[b].x - f[b] * next.x, cur[b].y - f[b] * next.y);
        d[(long)(k1 - b) * modes + mn] = next;
      }
  }
}

// the same on request: no later solve has added the sums up
__global__ __launch_bounds__(256) void final_test_kernel(RefineState rs) {
  __shared__ double2 s[256];
  double rr = 0.0, bb = 0.0;
  for (int i = (int)threadIdx.x; i < rs.nb; i += 256) {
    rr += rs.partials[2 * (long)i];
    bb += rs.partials[2 * (long)i + 1];
  }
  s[threadIdx.x] = make_double2(rr, bb);
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) s[threadIdx.x] = c_add(s[threadIdx.x], s[threadIdx.x + off]);
    __syncthreads();
  }
  if (threadIdx.x != 0 || !rs.ctl[3]) return;
  rs.norms[0] = s[0].x;
  rs.norms[1] = s[0].y;
  const int done = s[0].x <= rs.tol2 * s[0].y || s[0].x == 0.0;
  rs.ctl[0] = done;
  if (!done) rs.ctl[2] += 1;
  rs.ctl[3] = 0;
}

// the tridiagonal factors inv[k][mode] = 1 / (diag - inv[k - 1][mode]),
// diag = -(2 + 4 (sx2[m] + sy2[n])), of cols columns
__global__ __launch_bounds__(64) void factor_kernel(const double* __restrict__ sx2, const double* __restrict__ sy2,
                                                    int cols, int ny, int K, double* __restrict__ inv) {
  const long modes = (long)cols * ny;
  const long mn = (long)blockIdx.x * 64 + threadIdx.x;
  if (mn >= modes) return;
  const int n = (int)(mn / cols), m = (int)(mn - (long)n * cols);
  const double diag = -(2.0 + 4.0 * (sx2[m] + sy2[n]));
  double f = 0.0;
  for (int k = 0; k < K; ++k) {
    f = 1.0 / (diag - f);
    inv[(long)k * modes + mn] = f;
  }
}

unsigned mul_of(int d) { return d <= 1 ? 0u : (unsigned)(((1ull << 32) + (unsigned)d - 1) / (unsigned)d); }

// the fewest radices of 2..6 and 8 whose product is n (ties: the smallest sum);
// false if n has another prime factor
bool radices(int n, int* out, int* count) {
  static const int kR[] = {8, 6, 5, 4, 3, 2};
  int best[16], bn = 1000, bsum = 0, cur[16];
  auto rec = [&](auto&& self, int rem, int from, int depth, int sum) -> void {
    if (rem == 1) {
      if (depth < bn || (depth == bn && sum < bsum)) {
        bn = depth;
        bsum = sum;
        std::copy(cur, cur + depth, best);
      }
      return;
    }
    if (depth >= 10) return;
    for (int i = from; i < 6; ++i)
      if (rem % kR[i] == 0) {
        cur[depth] = kR[i];
        self(self, rem / kR[i], i, depth + 1, sum + kR[i]);
      }
  };
  rec(rec, n, 0, 0, 0);
  if (bn > kFftStages) return false;
  *count = bn;
  std::copy(best, best + bn, out);
  return true;
}

bool line_plan(int N, FftLine* f) {
  f->N = N;
  int r[16];
  if (!radices(N, r, &f->nst)) return false;
  int s = 1;
  for (int i = 0; i < f->nst; ++i) {
    f->radix[i] = r[i];
    f->mul_s[i] = mul_of(s);
    s *= r[i];
  }
  return true;
}

constexpr size_t kLdsMost = 160 * 1024 - 512;  // dynamic LDS of a block (gfx950: 160 KiB a CU)

size_t row_lds(const SpectralPlan& p) {
  return sizeof(double2) * ((size_t)p.fx.N + (p.full ? p.fy.N : 0) + 2 * (size_t)p.buf);
}
int row_threads(const SpectralPlan& p) { return p.full ? kRowThreads : 256; }

template <int kChunks, int kModes>
void tridiag_len(double2* w, const double* inv, int K, long modes, const RefineState& rs, hipStream_t st) {
  const int len = (K + kChunks - 1) / kChunks;
  const dim3 grid((unsigned)((modes + kModes - 1) / kModes + (rs.ctl ? 1 : 0))), blk(kChunks * kModes);
  if (len <= 4)
    hipLaunchKernelGGL((tridiag_kernel<kChunks, kModes, 4>), grid, blk, 0, st, w, inv, K, modes, rs);
  else if (len <= 8)
    hipLaunchKernelGGL((tridiag_kernel<kChunks, kModes, 8>), grid, blk, 0, st, w, inv, K, modes, rs);
  else if (len <= 16)
    hipLaunchKernelGGL((tridiag_kernel<kChunks, kModes, 16>), grid, blk, 0, st, w, inv, K, modes, rs);
  else
    hipLaunchKernelGGL((tridiag_kernel<kChunks, kModes, 32>), grid, blk, 0, st, w, inv, K, modes, rs);
}

}  // namespace

bool spectral_plan(int nx, int ny, int nz, SpectralPlan* p) {
  std::memset(p, 0, sizeof(*p));
  if (!line_plan(nx, &p->fx) || !line_plan(ny, &p->fy)) return false;
  p->K = nz - 1;
  p->hx = nx / 2 + 1;
  p->npair = (ny + 1) / 2;
  p->ldx = nx | 1;
  // whole planes while two buffers of the half spectrum (or of the packed
  // rows) and the twiddles fit in LDS
  const int whole = std::max(p->npair * p->ldx, ny * p->hx);
  if (sizeof(double2) * ((size_t)nx + ny + 2 * (size_t)whole) <= kLdsMost) {
    p->full = 1;
    p->pairs = p->npair;
    p->chunks = 1;
    p->buf = whole;
  } else {
    // row pairs and columns per block: about 1,000 points, so several blocks
    // share a CU
    p->pairs = std::max(1, std::min(p->npair, 1024 / nx));
    p->chunks = (p->npair + p->pairs - 1) / p->pairs;
    p->buf = p->pairs * std::max(p->ldx, 2 * p->hx);
    const int most = std::max(1, std::min(p->hx, 2048 / ny));
    p->col_chunks = (p->hx + most - 1) / most;
    p->cols = (p->hx + p->col_chunks - 1) / p->col_chunks;
    p->col_chunks = (p->hx + p->cols - 1) / p->cols;
    p->mul_cols = mul_of(p->cols);
    p->mul_cols_last = mul_of(p->hx - (p->col_chunks - 1) * p->cols);
  }
  p->mul_nx = mul_of(nx);
  p->mul_hx = mul_of(p->hx);
  p->mul_pairs = mul_of(p->pairs);
  p->mul_last = mul_of(p->npair - (p->chunks - 1) * p->pairs);
  return true;
}

int spectral_setup() {
  const void* k[] = {(const void*)rows_fwd_kernel<kRhsUnit>, (const void*)rows_fwd_kernel<kRhsRho64>,
                     (const void*)rows_fwd_kernel<kRhsFixed>, (const void*)rows_inv_kernel,
                     (const void*)cols_kernel<true>,
                     (const void*)cols_kernel<false>};
  for (const void* f : k)
    if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsMost) != hipSuccess) return -1;
  return 0;
}

void launch_factors(const double* sx2, const double* sy2, int cols, int ny, int K, double* inv, hipStream_t st) {
  const long modes = (long)cols * ny;
  hipLaunchKernelGGL(factor_kernel, dim3((unsigned)((modes + 63) / 64)), dim3(64), 0, st, sx2, sy2, cols, ny, K, inv);
}

void launch_spectral_solve(const SpectralPlan& p, const SpectralArgs& a, int in, double2* work, const double* inv,
                           const RefineState& rs, hipStream_t st) {
  const dim3 rows((unsigned)(p.K * p.chunks)), thr(row_threads(p));
  const size_t lds = row_lds(p);
  if (in == kRhsUnit)
    hipLaunchKernelGGL(rows_fwd_kernel<kRhsUnit>, rows, thr, lds, st, p, a, work);
  else if (in == kRhsRho64)
    hipLaunchKernelGGL(rows_fwd_kernel<kRhsRho64>, rows, thr, lds, st, p, a, work);
  else
    hipLaunchKernelGGL(rows_fwd_kernel<kRhsFixed>, rows, thr, lds, st, p, a, work);
  const size_t col_lds = sizeof(double2) * ((size_t)p.fy.N + 2 * (size_t)p.cols * p.fy.N);
  if (!p.full)
    hipLaunchKernelGGL(cols_kernel<true>, dim3((unsigned)(p.K * p.col_chunks)), dim3(256), col_lds, st, p, a.tw_y,
                       work);
  const long modes = (long)p.hx * p.fy.N;
  // chunks along z: 16 threads a mode for short columns of planes, 32 beyond
  if (p.K <= 64)
    tridiag_len<16, 8>(work, inv, p.K, modes, rs, st);
  else if (p.K <= 1024)
    tridiag_len<32, 8>(work, inv, p.K, modes, rs, st);
  else {
    hipLaunchKernelGGL(tridiag_serial_kernel, dim3((unsigned)((modes + 63) / 64)), dim3(64), 0, st, work, inv, p.K,
                       modes);
    if (rs.ctl) {  // the previous solve's test, which the chunked kernel's extra block takes
      hipLaunchKernelGGL(final_test_kernel, dim3(1), dim3(256), 0, st, rs);
      launch_fill_int(rs.ctl + 3, 1, 1, st);
      launch_fill_int(rs.ctl + 1, 1, 1, st);
    }
  }
  if (!p.full)
    hipLaunchKernelGGL(cols_kernel<false>, dim3((unsigned)(p.K * p.col_chunks)), dim3(256), col_lds, st, p, a.tw_y,
                       work);
  hipLaunchKernelGGL(rows_inv_kernel, rows, thr, lds, st, p, a.tw_x, a.tw_y, work, a.psi);
}

void launch_final_test(const RefineState& rs, hipStream_t st) {
  hipLaunchKernelGGL(final_test_kernel, dim3(1), dim3(256), 0, st, rs);
}

}  // namespace pic
