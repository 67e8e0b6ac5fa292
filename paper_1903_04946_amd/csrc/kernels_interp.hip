// kernels_interp.hip -- trigonometric interpolation of a grid wavefunction
// onto another uniform grid (Appendix B: wavefunctions on grids of different
// range and density are compared by trigonometric interpolation of the one
// on the sparser grid).
//
// Along one axis the interpolant of samples u_m (m = 0..n-1, x_m = lo + m dx,
// L = n dx) is u(x) = sum_k c_k exp(2 pi i k xi) with xi = (x - lo)/L and
// c_k = (1/n) sum_m u_m exp(-2 pi i k m/n), k over the symmetric band
// |k| < n/2; for even n the Nyquist coefficient enters as c_{n/2} cos(pi n xi),
// so real samples give a real interpolant and the grid points reproduce their
// samples.  Points outside [lo, lo + L) take the value zero (the wavefunction
// is taken to vanish outside the grid it was propagated on).
//
// The interpolant is linear in the samples: u(x_j) = sum_m W_jm u_m with the
// REAL matrix W_jm = (1 + 2 sum_{0<k<n/2} cos(2 pi k (xi_j - m/n)) [+ Nyquist])/n
// (the band is symmetric, so the sine terms cancel), and on a 3D grid the
// three axis matrices act in turn (z, then y, then x).  A complex state is
// then twice as many real columns: each axis is a real FP64 matrix product on
// the matrix cores, half the operations of the complex product with the
// matrix' (zero) imaginary part.  Rows of W outside the source box are zero,
// and the rows inside are one interval of j: only that interval is formed,
// multiplied and kept between the axes, and the rest of the destination is
// filled with zeros.
#include <algorithm>

#include "fft_core.hpp"
#include "internal.hpp"

namespace sop {
namespace {

// Wt[m][j - j0] for source sample m and destination point j in [j0, j0 + nj),
// columns nj..ldw-1 zero.  The position xi is computed without contraction, in
// the same order as the plain definition (dx_dst = (hi_dst - lo_dst)/n_dst,
// x = lo_dst + j dx_dst, xi = (x - lo)/(hi - lo)).  The phase 2 pi k (xi n - m)/n
// is reduced exactly: xi n = f_i + f_f (integer and fraction), and
// k (f_i - m) mod n is an integer r, stepped by additions mod n, leaving
// 2 pi (r + k f_f)/n with |r + k f_f| < 1.5 n.
__global__ void __launch_bounds__(128)
    k_interp_weights(double* __restrict__ Wt, int n, double lo, double hi, int nd, double lod,
                     double hid, int j0, int nj, int ldw) {
#pragma clang fp contract(off)
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  const int m = blockIdx.y;
  if (c >= ldw) return;
  double w = 0.0;
  if (c < nj) {
    const double dxd = (hid - lod) / nd;
    const double x = lod + (j0 + c) * dxd;
    const double xi = (x - lo) / (hi - lo);
    const double f = xi * n;
    const double fi = floor(f);
    const double ff = f - fi;
    const int d0 = (int)fi - m;  // integer part of xi n - m, |d0| <= n
    const int dm = d0 < 0 ? d0 + n : (d0 >= n ? d0 - n : d0);
    const int kmax = (n - 1) / 2;  // |k| < n/2
    double re = 0.0;
    int r = 0;
    for (int k = 1; k <= kmax; ++k) {
      r += dm;
      if (r >= n) r -= n;
      const double ph = (2.0 * 3.14159265358979323846) * (((double)r + k * ff) / n);
      double s, co;
      sincos_phase(ph, &s, &co);
      re += co;
    }
    re = 1.0 + 2.0 * re;
    if ((n & 1) == 0) {  // Nyquist: cos(pi (xi n - m)) = (-1)^d0 cos(pi ff)
      double s, co;
      sincos_phase(3.14159265358979323846 * ff, &s, &co);
      re += (d0 & 1) ? -co : co;
    }
    w = re / n;
  }
  Wt[(size_t)m * ldw + c] = w;
}

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int NT = 256;       // threads per workgroup, four waves
constexpr int BN = 128;       // real columns (64 complex) per workgroup
constexpr int BK = 16;        // source samples per LDS slab
constexpr uint32_t kOutside = 0xfffffff0u;  // a byte offset no buffer reaches

// Zeros at the destination points outside the box of intervals [j0, j0 + nj)
// of each axis, a row of the contiguous axis per workgroup and turn (a launch
// of its own: the same stores at the end of the last axis' workgroups held
// their LDS and registers and took longer, 342 against 192 + 97 us).
__global__ void __launch_bounds__(256) k_interp_zero(InterpZero g) {
  const int rows = g.n[0] * g.n[1] * g.S;
  const double2 z = make_double2(0.0, 0.0);
  for (int r = blockIdx.x; r < rows; r += gridDim.x) {
    const int y = r % g.n[1], x = (r / g.n[1]) % g.n[0];
    const bool inside = x >= g.j0[0] && x < g.j0[0] + g.nj[0] && y >= g.j0[1] &&
                        y < g.j0[1] + g.nj[1];
    double2* row = g.out + (size_t)r * g.n[2];
    for (int i = threadIdx.x; i < g.n[2]; i += 256)
      if (!inside || i < g.j0[2] || i >= g.j0[2] + g.nj[2]) row[i] = z;
  }
}

// One axis: C(j, col) = sum_m Wt[m][j] X(m, col) over the real columns `col`
// of the complex state (interleaved re, im), FP64, on v_mfma_f64_16x16x4.
//
// What bounds it: the FP64 matrix rate (75 TFLOP/s measured for the
// instruction alone, 64 cycles each); a wave's four samples issue TM * TN of
// them for (TM + TN) / 2 16-byte LDS reads, so LDS stays far from its limit.
// BM output rows by 128 real columns per workgroup, waves of (16 TM) x (16 TN);
// slabs of BK samples go through two LDS buffers, the next slab's global
// loads in flight during the current one's products.
// A tile's operand lanes hold two neighbouring rows (columns) of each 32, so
// that every LDS read is a contiguous 16 bytes a lane and an output lane
// holds whole complex values.
// KROW: X is contiguous along m (the axis is the contiguous one): X(m, (r, c))
// = component c of state[r][m], and the slab is transposed on its way to LDS.
// The workgroups of one column panel (nm of them) are 8 apart in the linear
// block index: consecutive workgroups go to the 8 XCDs in turn, so a panel's
// workgroups share an XCD's L2 and the panel is read from memory once.
// Measured for 128^3 -> 256^3 x 3, the box sqrt 2 wider (181 of 256 points an
// axis inside): 109, 142 and 192 us for z, y and x (44-51 TFLOP/s, the matrix
// cores busy 57-68% of the time) where the dense complex product on the
// vector units took 268, 518 and 1007; the whole call 1585 -> 515 us, 97 of
// them the zeros.  Persistent workgroups that fetch the next tile's first
// slab during the last products, operands read one step ahead, and 96-row
// tiles all took the same times.
template <int BM, int TM, int TN, bool KROW>
__global__ void __launch_bounds__(NT, 2) k_interp_axis(InterpAxis g) {
  constexpr int LA = BM + 2, LB = BN + 2;  // padded rows: 16-byte shifts between samples
  constexpr int WN = BN / (16 * TN);       // waves along the columns
  static_assert((BM / (16 * TM)) * WN == 4, "four waves cover the tile");
  __shared__ __align__(16) double As[2][BK * LA];
  __shared__ __align__(16) double Bs[2][BK * LB];
  const int t = threadIdx.x, l = t & 63, wv = t >> 6;
  const int xcd = blockIdx.x & 7, kq = blockIdx.x >> 3;
  const int pan = (kq / g.nm) * 8 + xcd;  // column panel
  if (pan >= g.npan * g.batch) return;
  const int b = pan / g.npan;
  const int c0 = pan % g.npan * (BN / 2);  // first complex column
  const int m0 = kq % g.nm * BM;           // first output row
  // 16-byte buffer loads; columns past the last take an offset outside the
  // buffer's extent and read zero, without a branch around each load
  const auto rx = rsrc((const cx<double>*)g.X + (size_t)b * g.bsx, g.xel);
  const auto rw = rsrc((const cx<double>*)g.Wt, (uint32_t)((size_t)g.K * g.ldw / 2));
  constexpr int QA = BK * BM / (2 * NT), QB = BK * BN / (2 * NT);
  static_assert(QA >= 1 && QB >= 1, "slab loads");
  sop_u32x4 ra[QA], rb[QB];
  uint32_t oa[QA], ob[QB];  // byte offsets of slab 0
  int la[QA], lb[QB];       // LDS slots (doubles)
#pragma unroll
  for (int q = 0; q < QA; ++q) {
    const int e = t + NT * q;
    const int k = e / (BM / 2), m = (e % (BM / 2)) * 2;
    oa[q] = (uint32_t)(k * g.ldw + m0 + m) * 8u;
    la[q] = k * LA + m;
  }
#pragma unroll
  for (int q = 0; q < QB; ++q) {
    const int k = KROW ? t % BK : t / (BN / 2) + (2 * NT / BN) * q;
    const int c = KROW ? t / BK + (NT / BK) * q : t % (BN / 2);
    const int cc = c0 + c;
    ob[q] = cc < g.N ? (KROW ? (uint32_t)cc * (uint32_t)g.K + k
                             : (uint32_t)k * (uint32_t)g.ldx + cc) * 16u
                     : kOutside;
    lb[q] = k * LB + 2 * c;
  }
  const uint32_t sa = (uint32_t)BK * g.ldw * 8u;  // bytes a slab
  const uint32_t sb = (KROW ? (uint32_t)BK : (uint32_t)BK * (uint32_t)g.ldx) * 16u;
  auto fetch = [&](uint32_t k) {  // slab k
#pragma unroll
    for (int q = 0; q < QA; ++q)
      ra[q] = __builtin_amdgcn_raw_buffer_load_b128(rw, (int)(oa[q] + k * sa), 0, 0);
#pragma unroll
    for (int q = 0; q < QB; ++q)
      rb[q] = __builtin_amdgcn_raw_buffer_load_b128(
          rx, (int)(ob[q] == kOutside ? kOutside : ob[q] + k * sb), 0, 0);
  };
  auto put = [&](int buf) {
#pragma unroll
    for (int q = 0; q < QA; ++q) *reinterpret_cast<sop_u32x4*>(&As[buf][la[q]]) = ra[q];
#pragma unroll
    for (int q = 0; q < QB; ++q) *reinterpret_cast<sop_u32x4*>(&Bs[buf][lb[q]]) = rb[q];
  };
  const int li = l & 15, lk = l >> 4;
  const int wm = (wv / WN) * (16 * TM), wn = (wv % WN) * (16 * TN);
  f64x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
  fetch(0);
  put(0);
  __syncthreads();
  int buf = 0;
  const int slabs = g.K / BK;
  for (int k0 = 0; k0 < slabs; ++k0) {
    const bool more = k0 + 1 < slabs;
    if (more) fetch(k0 + 1);
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      double a[TM], x[TN];
#pragma unroll
      for (int i = 0; i < TM; i += 2) {
        const f64x2 v =
            *reinterpret_cast<const f64x2*>(&As[buf][(kk + lk) * LA + wm + 16 * i + 2 * li]);
        a[i] = v.x;
        a[i + 1] = v.y;
      }
#pragma unroll
      for (int j = 0; j < TN; j += 2) {
        const f64x2 v =
            *reinterpret_cast<const f64x2*>(&Bs[buf][(kk + lk) * LB + wn + 16 * j + 2 * li]);
        x[j] = v.x;
        x[j + 1] = v.y;
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], x[j], acc[i][j], 0, 0, 0);
    }
    if (more) put(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }
  // lane l, register r of a 16 x 16 tile: row 4 r + l / 16, column l % 16;
  // tile (i, j) holds rows 32 (i / 2) + 2 row + i % 2 and real columns
  // 32 (j / 2) + 2 col + j % 2 of the wave
  double2* C = g.C + (size_t)b * g.bsc;
#pragma unroll
  for (int j = 0; j < TN; j += 2) {
    const int cc = c0 + wn / 2 + 8 * j + li;  // complex column
    if (cc >= g.N) continue;
    const size_t co = KROW ? (size_t)cc * g.ldc
                           : (size_t)(cc / g.cdiv) * g.crow + (size_t)(cc % g.cdiv);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + wm + 32 * (i / 2) + 2 * (4 * r + lk) + i % 2;
        if (m < g.M)
          C[co + (KROW ? (size_t)m : (size_t)m * g.ldc)] =
              make_double2(acc[i][j][r], acc[i][j + 1][r]);
      }
  }
}

// 1D grids (at most two surfaces, four real columns): the product is a pass
// over the matrix, one read of each entry.  64 destination points by 16
// slices of the samples per workgroup, neighbouring points on neighbouring
// lanes; the slices are summed through LDS in a fixed order.
template <int S>
__global__ void __launch_bounds__(1024)
    k_interp_rows(const double* __restrict__ Wt, int ldw, int n, int nj,
                  const double2* __restrict__ X, double2* __restrict__ out, int nd) {
  __shared__ double2 red[16][S][64];
  const int c = threadIdx.x & 63, sl = threadIdx.x >> 6;
  const int j = blockIdx.x * 64 + c;  // below ldw: its columns past nj are zero
  double2 a[S];
#pragma unroll
  for (int s = 0; s < S; ++s) a[s] = make_double2(0.0, 0.0);
#pragma unroll 8
  for (int m = sl; m < n; m += 16) {
    const double w = Wt[(size_t)m * ldw + j];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const double2 x = X[(size_t)s * n + m];
      a[s].x = fma(w, x.x, a[s].x);
      a[s].y = fma(w, x.y, a[s].y);
    }
  }
#pragma unroll
  for (int s = 0; s < S; ++s) red[sl][s][c] = a[s];
  __syncthreads();
  if (sl < S && j < nj) {
    double2 v = make_double2(0.0, 0.0);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      v.x += red[i][sl][c].x;
      v.y += red[i][sl][c].y;
    }
    out[(size_t)sl * nd + j] = v;
  }
}

template <int BM, int TM, int TN>
hipError_t launch_axis(hipStream_t s, InterpAxis g, bool krow) {
  g.nm = (g.M + BM - 1) / BM;
  g.npan = (g.N + BN / 2 - 1) / (BN / 2);
  const long long panels = (long long)g.npan * g.batch;
  const long long tiles = (panels + 7) / 8 * 8 * g.nm;
  if (tiles > 0x7fffffffLL || g.ldw < g.nm * BM || g.K % BK != 0) return hipErrorInvalidValue;
  // a batch entry's extent, with 32-bit byte offsets
  const long long xel = krow ? (long long)g.N * g.K : (long long)(g.K - 1) * g.ldx + g.N;
  if (xel >= (1LL << 28) || (long long)g.K * g.ldw >= (1LL << 29)) return hipErrorInvalidValue;
  g.xel = (uint32_t)xel;
  const unsigned blocks = (unsigned)tiles;
  if (krow)
    hipLaunchKernelGGL((k_interp_axis<BM, TM, TN, true>), dim3(blocks), dim3(NT), 0, s, g);
  else
    hipLaunchKernelGGL((k_interp_axis<BM, TM, TN, false>), dim3(blocks), dim3(NT), 0, s, g);
  return hipGetLastError();
}

}  // namespace

void interp_inside(int n, double lo, double hi, int nd, double lod, double hid, int* j0, int* nj) {
#pragma clang fp contract(off)
  (void)n;
  // xi does not decrease with j, so the points with 0 <= xi < 1 are an interval
  int first = nd, last = -1;
  const double dxd = (hid - lod) / nd;
  for (int j = 0; j < nd; ++j) {
    const double x = lod + j * dxd;
    const double xi = (x - lo) / (hi - lo);
    if (xi >= 0.0 && xi < 1.0) {
      if (first == nd) first = j;
      last = j;
    }
  }
  *j0 = last < 0 ? 0 : first;
  *nj = last < 0 ? 0 : last - first + 1;
}

hipError_t interp_weights(hipStream_t s, double* Wt, int n, double lo, double hi, int nd,
                          double lod, double hid, int j0, int nj, int ldw) {
  if (n < 1 || n > 65535 || nd < 1 || nj < 1 || ldw < nj) return hipErrorInvalidValue;
  dim3 grid((ldw + 127) / 128, n);
  hipLaunchKernelGGL(k_interp_weights, grid, dim3(128), 0, s, Wt, n, lo, hi, nd, lod, hid, j0,
                     nj, ldw);
  return hipGetLastError();
}

hipError_t interp_axis(hipStream_t s, const InterpAxis& g, bool krow) {
  if (g.M < 1 || g.N < 1 || g.K < 1 || g.batch < 1) return hipErrorInvalidValue;
  // 128 rows where they pad M no more than smaller tiles do (fewer reads of the
  // columns), 32 for up to 32 points, else 64
  const int p32 = (g.M + 31) / 32, p64 = (g.M + 63) / 64 * 2, p128 = (g.M + 127) / 128 * 4;
  if (p128 <= p64 && p128 <= p32) return launch_axis<128, 4, 4>(s, g, krow);
  if (p64 <= p32 || g.M > 32) return launch_axis<64, 2, 4>(s, g, krow);
  return launch_axis<32, 2, 2>(s, g, krow);
}

hipError_t interp_rows(hipStream_t s, const double* Wt, int ldw, int n, int S, int nj,
                       const double2* X, double2* out, int nd) {
  if (n < 1 || nj < 1 || ldw % 64 != 0 || ldw < nj) return hipErrorInvalidValue;
  const dim3 grid((nj + 63) / 64);
  if (S == 1)
    hipLaunchKernelGGL(k_interp_rows<1>, grid, dim3(1024), 0, s, Wt, ldw, n, nj, X, out, nd);
  else if (S == 2)
    hipLaunchKernelGGL(k_interp_rows<2>, grid, dim3(1024), 0, s, Wt, ldw, n, nj, X, out, nd);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t interp_zero(hipStream_t s, const InterpZero& g) {
  const long long rows = (long long)g.n[0] * g.n[1] * g.S;
  if (rows < 1 || rows > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_interp_zero, dim3((unsigned)std::min(rows, 65536LL)), dim3(256), 0, s, g);
  return hipGetLastError();
}

}  // namespace sop
