// passes_3d.hpp -- pencil schedules and the bodies of the pass kinds of the
// 3D executor, as device functions of one workgroup tile.  The kernels of a
// single plan (kernels_3d.hip) and of a batch of plans (kernels_batch3d.hip)
// wrap the same bodies, so both compute identical values.
//
// The kinetic propagator of a separable T(p) = sum_d p_d^2 / (2 m_d) factors
// over the axes: exp(-i tau T / hbar) = K_z K_y K_x with the commuting
// one-dimensional actions K_d = F_d^-1 diag(f_d) F_d along axis d (Sec.
// "Dynamic Fourier method": the kinetic action is diagonal in the momentum
// representation, and both it and the FFT factor over the axes).  A substep
// (one potential action followed by one kinetic action) is therefore three
// passes over psi[s][z][y][x], each taking the state from and back to the
// position representation:
//   z-pass : potential unitary(ies) -> forward FFT z -> f_z -> inverse FFT z
//            (all S surfaces of a tile of x-columns: the S x S matvec of
//            Sec. "Molecular Hamiltonian in the diabatic basis" runs in
//            registers);
//   y-pass : forward FFT y -> f_y -> inverse FFT y;
//   x-pass : forward FFT x -> f_x -> inverse FFT x.
// Where the whole xy plane fits in LDS the y- and x-passes run as one plane
// pass.  The per-axis factor f_d(k) = exp(-i tau hbar kappa_k^2 / (2 m_d)) / n_d
// carries the 1/n_d of the unnormalised inverse transform.
#pragma once

#include <type_traits>

#include "eigen.hpp"
#include "fft_core.hpp"
#include "internal.hpp"

namespace sop {
namespace s3d {

using Z32 = Sched<32, 8, RList<8, 4>, RList<4, 8>, 8, 4>;
using Z48 = Sched<48, 12, RList<12, 4>, RList<4, 12>, 12, 4>;
using Z64 = Sched<64, 8, RList<8, 8>, RList<8, 8>, 8, 8>;
using Z128 = Sched<128, 8, RList<8, 4, 4>, RList<4, 4, 8>, 8, 4>;
using Z256 = Sched<256, 8, RList<8, 8, 4>, RList<4, 8, 8>, 8, 4>;

// Schedules of the single-pencil y and x passes: sixteen values per thread
// where that saves an LDS exchange.
template <class SC>
struct XYSched {
  using type = SC;
};
template <>
struct XYSched<Z128> {
  using type = Sched<128, 16, RList<16, 8>, RList<8, 16>, 16, 8>;
};
template <>
struct XYSched<Z256> {
  using type = Sched<256, 16, RList<16, 16>, RList<16, 16>, 16, 16>;
};

// Columns per tile of the y-pass: at least a full wave per block and
// 128-byte contiguous row segments.
template <class SC, typename T>
constexpr int cols() {
  constexpr int seg = 128 / (int)sizeof(cx<T>);
  return SC::TPC * seg >= 64 ? seg : 64 / SC::TPC;
}

// Rows per x-pass block: about 128 threads, and a divisor of N.
template <class XS>
constexpr int xrows() {
  int r = XS::TPC >= 16 ? 8 : 128 / XS::TPC;
  while (XS::N % r != 0) r /= 2;
  return r;
}

// Column width of the potential-table tiles (and of the default z-pass tile):
// 16 in both precisions, 256-byte FP64 and 128-byte FP32 segments of psi.
constexpr int kTableCols = 16;

}  // namespace s3d

// Complex entries of one axis block of the twiddle and factor tables (in FP32
// the (rounded, residue) pairs of Split<float>).
template <typename T, int N>
constexpr int axis_block() {
  return N * Split<T>::rep;
}

// LDS of the y-pass tiles (C columns) and of the x-pass tiles (ROWS rows):
// the exchange area and two staged axis blocks (twiddles, factor).  The
// z-pass reads its twiddles and factor from global memory: with the
// potential's table reads in flight, staging them measured slower (57.2
// against 54.8 us a pass for 128^3 x 3 FP64), while it saves 4-5% on the
// y-, x- and plane passes.
template <typename T, int N>
constexpr size_t y_lds_elems(int C) {
  return (size_t)C * N + 2 * axis_block<T, N>();
}
template <typename T, int N>
constexpr size_t x_lds_elems(int ROWS) {
  return (size_t)ROWS * (N + N / 16) + 2 * axis_block<T, N>();
}

// Copies nb axis blocks (src[b], axis_block entries each) into LDS at dst,
// every thread of the block striding over them.  The y-, x- and plane passes
// stage their twiddles and kinetic factors this way before loading their
// pencils: every later read of them is an LDS read instead of a dependent
// global load in the middle of the transform.  Every transform starts with a
// stage that uses no twiddles, followed by an LDS exchange whose barrier
// orders these writes before the first read.
// `lane` and `nt` are the thread's index in the tile and the tile's thread
// count.
template <typename T, int N, int NB>
__device__ __forceinline__ void stage_blocks(cx<T>* dst, const cx<T>* const (&src)[NB], int lane,
                                             int nt) {
  constexpr int A = axis_block<T, N>();
  for (int i = lane; i < A; i += nt) {
#pragma unroll
    for (int b = 0; b < NB; ++b) dst[b * A + i] = src[b][i];
  }
}

// What a pass does along its axis after its pointwise work:
//   AX_NONE: nothing (z-pass carrying only potential actions);
//   AX_KIN : forward FFT -> per-axis kinetic factor -> inverse FFT.
enum { AX_NONE = 0, AX_KIN = 1 };

// v (forward-transformed, radix-RL ownership) *= f[k] (conjugated factor
// when conj): the kinetic factor of one axis (a split block in FP32).
template <typename T, class SC, int P>
__device__ __forceinline__ void axis_phase(cx<T> (*v)[SC::E], const cx<T>* __restrict__ f,
                                           T csign, int t) {
#pragma unroll
  for (int q = 0; q < SC::E; ++q) {
    const Fac<T> w = load_fac(f, own_idx<SC::N, SC::E, SC::RL>(t, q), csign);
#pragma unroll
    for (int p = 0; p < P; ++p) v[p][q] = fmul(v[p][q], w);
  }
}

// ---------------------------------------------------------------- eigen form
// cache-policy bits of a buffer load: non-temporal
constexpr int kCpolNT = 2;

// The functions of the eigen form fix their fused operations themselves (no
// contraction left to the compiler): several kernels inline them, and a
// state's result must not depend on which one ran it.
template <typename T, int S>
__device__ __forceinline__ void rotation_from_slots(const cx<T>* q, T (&R)[S][S]) {
#pragma clang fp contract(off)
  if constexpr (S == 2) {
    const T c = q[0].re, s = q[0].im;
    R[0][0] = c;
    R[0][1] = -s;
    R[1][0] = s;
    R[1][1] = c;
  } else {
    const T w = q[0].re, x = q[0].im, y = q[1].re, z = q[1].im;
    const T x2 = x + x, y2 = y + y, z2 = z + z;
    const T wx = w * x2, wy = w * y2, wz = w * z2;
    R[0][0] = fma(-z2, z, fma(-y2, y, (T)1));
    R[0][1] = fma(x2, y, -wz);
    R[0][2] = fma(x2, z, wy);
    R[1][0] = fma(x2, y, wz);
    R[1][1] = fma(-z2, z, fma(-x2, x, (T)1));
    R[1][2] = fma(y2, z, -wx);
    R[2][0] = fma(x2, z, -wy);
    R[2][1] = fma(y2, z, wx);
    R[2][2] = fma(-y2, y, fma(-x2, x, (T)1));
  }
}

// The eigen-form potential action at one point: R, and exp(-i tau lam) per
// eigenvalue, from the point's slots; applied to a state in FP64.
template <int S>
struct EigPoint {
  double R[S][S], cs[S], sn[S];
  __device__ __forceinline__ void form(const cx<double> (&sl)[eig_slots(S)], double tau) {
#pragma clang fp contract(off)
    rotation_from_slots<double, S>(sl, R);
    const double lam[3] = {sl[S == 3 ? 2 : 1].re, sl[S == 3 ? 2 : 1].im,
                           S == 3 ? sl[eig_slots(S) - 1].re : 0.0};
#pragma unroll
    for (int k = 0; k < S; ++k) sincos_phase(tau * lam[k], &sn[k], &cs[k]);
  }
  // gamma = R^T psi, gamma_k *= exp(-i tau lam_k), psi = R gamma, rounded once
  template <typename T>
  __device__ __forceinline__ void apply(cx<T> (&w)[S]) const {
#pragma clang fp contract(off)
    cx<double> g[S];
#pragma unroll
    for (int k = 0; k < S; ++k) {
      double re = R[0][k] * (double)w[0].re, im = R[0][k] * (double)w[0].im;
#pragma unroll
      for (int i = 1; i < S; ++i) {
        re = fma(R[i][k], (double)w[i].re, re);
        im = fma(R[i][k], (double)w[i].im, im);
      }
      // (re + i im) (cs - i sn)
      g[k] = cx<double>{fma(re, cs[k], im * sn[k]), fma(im, cs[k], -(re * sn[k]))};
    }
#pragma unroll
    for (int i = 0; i < S; ++i) {
      double re = R[i][0] * g[0].re, im = R[i][0] * g[0].im;
#pragma unroll
      for (int k = 1; k < S; ++k) {
        re = fma(R[i][k], g[k].re, re);
        im = fma(R[i][k], g[k].im, im);
      }
      w[i] = cx<T>{(T)re, (T)im};
    }
  }
};

// The packed entries of V0 + s D at points of one grid (the entries of D that
// are zero everywhere, clear in mask, come from descriptors of no extent).
template <int S>
struct DrivenRead {
  static constexpr int NE = S * (S + 1) / 2;
  const DrivenV& d;
  int64_t npts;
  double s;
  __device__ __forceinline__ void load(double (&v0)[NE], double (&v1)[NE], uint32_t pt) const {
    const uint32_t bytes = (uint32_t)npts * 8u;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const auto r0 = __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(d.v0 + e * npts),
                                                        (short)0, (int)bytes, 0x00020000);
      const auto r1 = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<double*>(d.d + e * npts), (short)0, (d.mask >> e) & 1 ? (int)bytes : 0,
          0x00020000);
      v0[e] = __builtin_bit_cast(
          double, __builtin_amdgcn_raw_buffer_load_b64(r0, (int)(pt * 8u), 0, 0));
      v1[e] = __builtin_bit_cast(
          double, __builtin_amdgcn_raw_buffer_load_b64(r1, (int)(pt * 8u), 0, 0));
    }
  }
  __device__ __forceinline__ void slots(const double (&v0)[NE], const double (&v1)[NE],
                                        cx<double> (&sl)[eig_slots(S)]) const {
    double A[S][S], R[S][S];
    int e = 0;
#pragma unroll
    for (int i = 0; i < S; ++i)
#pragma unroll
      for (int j = i; j < S; ++j, ++e) A[i][j] = A[j][i] = v0[e] + s * v1[e];
    jacobi_sym<S>(A, R);
    eig_form_slots<S>(A, R, sl);
  }
};

// On FP64 grids of 256 points a state of two or three surfaces (537, 805 MB) is
// beyond the last-level cache (256 MB), and little of the z-pass's output is
// left there for the y-pass: the z-pass stores and the y-pass loads it with the
// non-temporal hint, which spares the y-pass the write-back of what it evicts.
// us a pass without -> with: 256^3 x 2 y 194 -> 175, z 313, x 201 both (a TJ-6
// step 6.60 -> 6.41 ms); x 3 y 291 -> 281, z 548 -> 546, x 303 -> 310 (10.68 ->
// 10.65 ms).  On the z-pass's loads, and on the y- and x-passes' stores and the
// x-pass's loads, it gains nothing.  One surface (268 MB) partly stays, and
// loses with the hint (3.06 -> 3.14 ms a TJ-6 step).
template <typename T, int N, int S>
constexpr int kStateCpol = N >= 256 && S >= 2 && sizeof(T) == 8 ? kCpolNT : 0;

// ---------------------------------------------------------------- z-pass
// Potential tables are stored per tile of TC x-columns: for table u, tile
// (y, x / TC) holds [z][entry][x % TC] contiguously, N * NE * TC complex, so
// a tile reads its table as one contiguous stream.  The pass tile is C
// columns wide (C divides TC); block (bx, by) owns columns bx*C .. bx*C+C-1
// of row y = by.  `psi` is one state [S][N^3]; `fz` the z factor of the
// kinetic set (AX_KIN only).
//
// Table entries are cx<T>, in FP32 the pairs (rounded, residue) of
// Split<float> (each entry's index doubled).  `lane` (here and in the y- and
// x-pass bodies) is the thread's index in the tile, threadIdx.x unless a
// persistent caller passes it through opaque() so that the compiler does not
// keep every lane-derived offset live across its work loop.  `src` (here and
// there): where the pass reads the state, psi itself when NULL (in place);
// the pass always writes psi.
//
// EQ (S = 2, 3): `vexp` is instead the one compact eigen-form table, FP64 in
// both precisions (eig_slots(S) complex double slots per point, same tile
// layout), and `taus` the tau of each coefficient; a potential action is
// psi <- R exp(-i tau lam) R^T psi in registers, and the two actions at a
// step boundary share one load, one pair of rotations and one phase
// (psi <- R exp(-i (tau_1 + tau_2) lam) R^T psi: the same operator, rounded
// once).  The action is computed in FP64 in both precisions: an FP32 state
// is widened, rotated and phased in FP64 and rounded once, so the FP32 form
// carries no rounded potential operator.
template <typename T, class SC, int S, int C, int TC, int AX, bool EQ = false>
__device__ __forceinline__ void zpass_body(cx<T>* __restrict__ psi,
                                           const void* __restrict__ vexp, int nv, int iv0,
                                           int iv1, int conj, const cx<T>* __restrict__ tw,
                                           const cx<T>* __restrict__ fz, cx<T>* lds, int bx,
                                           int by, const double* __restrict__ taus = nullptr,
                                           int lane = (int)threadIdx.x,
                                           const cx<T>* src = nullptr) {
  static_assert(TC % C == 0, "pass tile must divide the table tile");
  static_assert(!EQ || S >= 2, "eigen form: two or three surfaces");
  constexpr int N = SC::N, E = SC::E, NE = EQ ? eig_slots(S) : S * (S + 1) / 2;
  const int col = lane % C, t = lane / C;
  const int x = bx * C + col, y = by;
  constexpr uint32_t plane = (uint32_t)N * N;
  constexpr int64_t npts = (int64_t)plane * N;
  constexpr uint32_t tile = (uint32_t)N * NE * TC;
  const uint32_t off0 = (uint32_t)y * N + x;
  const int tx = (C == TC) ? bx : (bx * C) / TC;            // table tile
  const int tcol = (C == TC) ? col : (bx * C) % TC + col;   // column within it
  const size_t tbase = ((size_t)y * (N / TC) + tx) * tile;
  const LayStrided lay{col, 0, C};  // one surface at a time through LDS
  cx<T> v[S][E];
  const cx<T>* const in = src ? src : psi;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const auto rs = rsrc(in + s * npts, (uint32_t)npts);
#pragma unroll
    for (int q = 0; q < E; ++q) v[s][q] = ld<T>(rs, own_idx<N, E, SC::RF>(t, q) * plane + off0);
  }
  const T csign = conj ? (T)-1 : (T)1;
  if constexpr (EQ) {
    if (nv >= 1) {
      const auto rq = rsrc((const cx<double>*)vexp + tbase, tile);
      // two actions at a step boundary: exp(-i tau_2 lam) exp(-i tau_1 lam)
      // = exp(-i (tau_1 + tau_2) lam), one phase per eigenvalue
      const double tab = (double)csign * (taus[iv0] + (nv >= 2 ? taus[iv1] : 0.0));
#pragma unroll
      for (int q = 0; q < E; ++q) {
        const uint32_t pt = (uint32_t)own_idx<N, E, SC::RF>(t, q) * (NE * TC) + tcol;
        cx<double> sl[NE];
#pragma unroll
        for (int e = 0; e < NE; ++e) {
          // an eigen table larger than the last-level cache (256^3: 1.07 GB)
          // is read with the non-temporal hint: read once a pass, it would
          // only evict the state from the caches
          const sop_u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(
              rq, (int)((pt + e * TC) * 16u), 0, N >= 256 ? kCpolNT : 0);
          sl[e] = __builtin_bit_cast(cx<double>, w);
        }
        EigPoint<S> ep;
        ep.form(sl, tab);
        cx<T> w[S];
#pragma unroll
        for (int s = 0; s < S; ++s) w[s] = v[s][q];
        ep.apply(w);
#pragma unroll
        for (int s = 0; s < S; ++s) v[s][q] = w[s];
      }
    }
  } else {
    constexpr int REP = Split<T>::rep;
    auto vact = [&](int iv) {
      const auto ru = rsrc((const cx<T>*)vexp + ((size_t)iv * NE * npts + tbase) * REP,
                           tile * REP);
#pragma unroll
      for (int q = 0; q < E; ++q) {
        const uint32_t pt = (uint32_t)own_idx<N, E, SC::RF>(t, q) * (NE * TC) + tcol;
        Fac<T> u[NE];
#pragma unroll
        for (int e = 0; e < NE; ++e) u[e] = ldfac<T>(ru, pt + e * TC, csign);
        cx<T> w[S];
#pragma unroll
        for (int s = 0; s < S; ++s) w[s] = v[s][q];
        apply_u_fac<T, S>(w, u);
#pragma unroll
        for (int s = 0; s < S; ++s) v[s][q] = w[s];
      }
    };
    if (nv >= 1) vact(iv0);
    if (nv >= 2) vact(iv1);
  }
  if constexpr (AX == AX_KIN) {
#pragma unroll
    for (int s = 0; s < S; ++s) fft_forward<SC, 1>(v + s, lds, lay, tw, t);
    axis_phase<T, SC, S>(v, fz, csign, t);
#pragma unroll
    for (int s = 0; s < S; ++s) fft_inverse<SC, 1>(v + s, lds, lay, tw, t);
  }
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const auto rs = rsrc(psi + s * npts, (uint32_t)npts);
#pragma unroll
    for (int q = 0; q < E; ++q)
      st<kStateCpol<T, N, S>>(rs, own_idx<N, E, SC::RF>(t, q) * plane + off0, v[s][q]);
  }
}

// ---------------------------------------------------------------- z tile
// The z-pass with a potential action in eigen form on grids of 32, 48 and 64
// points, for `ns` states of one plan: tile of C columns, NT threads.  The
// action's work is spread over all threads by points (C N / NT each), handed
// over in LDS, and the transforms are then a wave or half of one per surface
// (C * TPC threads), which needs no further barrier and stores its pencils.
// R and the phases of a point are formed once for all states.
// On these grids the z-pass is a chain of FP64 instructions, not traffic: with
// eight (48: twelve) points and all surfaces in each of a wave's lanes
// (zpass_body) a 32^3 x 3 pass has one wave on each compute unit, issuing
// about 350 instructions a point and surface set.  us a pass, one FP64
// state, zpass_body -> now: 32^3 x 3: 8.4 -> 4.5, 48^3 x 2: 9.9 -> 6.6, 64^3 x
// 3: 13.2 -> 9.8.  From 128 points on the pass is bound by memory: zpass_body.
// The same operations as zpass_body (EQ, AX_KIN) in the same order.
template <typename T, class SC, int S, int C, int NT, int AX = AX_KIN, bool DRV = false>
__device__ __forceinline__ void ztile_body(cx<T>* __restrict__ psi, int ns,
                                           const cx<double>* __restrict__ eig, double tau,
                                           int conj, const cx<T>* __restrict__ tw,
                                           const cx<T>* __restrict__ fz, cx<T>* lds, int bx,
                                           int by, const cx<T>* src, const DrivenV& drv = {}) {
  constexpr int N = SC::N, E = SC::E, NE = eig_slots(S), TC = s3d::kTableCols;
  constexpr int FT = C * SC::TPC;  // threads of one surface's transforms
  static_assert(64 % FT == 0 && NT >= FT * S && (C * N) % NT == 0 && TC % C == 0, "tile");
  constexpr int PP = C * N / NT;  // points per thread
  constexpr uint32_t plane = (uint32_t)N * N;
  constexpr int64_t npts = (int64_t)plane * N;
  constexpr uint32_t tile = (uint32_t)N * NE * TC;
  const int lane = (int)threadIdx.x;
  const uint32_t off0 = (uint32_t)by * N + bx * C;
  const size_t tbase = ((size_t)by * (N / TC) + (bx * C) / TC) * tile;
  const int tcol = (bx * C) % TC + lane % C;
  const T csign = conj ? (T)-1 : (T)1;
  cx<double> sl[PP][NE];
  [[maybe_unused]] const DrivenRead<S> dr{drv, npts, DRV ? *drv.s : 0.0};
  [[maybe_unused]] double a0[PP][S * (S + 1) / 2], a1[PP][S * (S + 1) / 2];
#pragma unroll
  for (int i = 0; i < PP; ++i) {
    const uint32_t z = lane / C + i * (NT / C);
    if constexpr (DRV) {
      dr.load(a0[i], a1[i], z * plane + off0 + lane % C);
    } else {
      const auto rq = rsrc(eig + tbase, tile);
#pragma unroll
      for (int e = 0; e < NE; ++e) sl[i][e] = ld<double>(rq, (z * NE + e) * TC + tcol);
    }
  }
  cx<T> w[PP][S];
  auto fetch = [&](int m) {  // the thread's points of state m
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const auto rs = rsrc((src ? src : psi) + ((size_t)m * S + s) * npts, (uint32_t)npts);
#pragma unroll
      for (int i = 0; i < PP; ++i)
        w[i][s] = ld<T>(rs, (uint32_t)(lane / C + i * (NT / C)) * plane + off0 + lane % C);
    }
  };
  fetch(0);  // arrives while R and the phases are formed
  const int wv = lane / FT, l = lane % FT, col = l % C, t = l / C;
  EigPoint<S> ep[PP];
#pragma unroll
  for (int i = 0; i < PP; ++i) {
    if constexpr (DRV) dr.slots(a0[i], a1[i], sl[i]);
    ep[i].form(sl[i], (double)csign * tau);
  }
  for (int m = 0; m < ns; ++m) {
    cx<T>* const out = psi + (size_t)m * S * npts;
    if (m > 0) fetch(m);
    if constexpr (AX == AX_NONE) {
#pragma unroll
      for (int i = 0; i < PP; ++i) ep[i].apply(w[i]);
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const auto rs = rsrc(out + s * npts, (uint32_t)npts);
#pragma unroll
        for (int i = 0; i < PP; ++i)
          st(rs, (uint32_t)(lane / C + i * (NT / C)) * plane + off0 + lane % C, w[i][s]);
      }
      continue;
    }
    if (m > 0) __syncthreads();  // the previous state's transforms are done with LDS
#pragma unroll
    for (int i = 0; i < PP; ++i) {
      ep[i].apply(w[i]);
#pragma unroll
      for (int s = 0; s < S; ++s) lds[s * (N * C) + lane + i * NT] = w[i][s];
    }
    __syncthreads();
    if (wv < S) {
      cx<T>* const area = lds + wv * (N * C);
      const LayStrided lay{col, 0, C};
      cx<T> v[1][E];
#pragma unroll
      for (int q = 0; q < E; ++q) v[0][q] = area[own_idx<N, E, SC::RF>(t, q) * C + col];
      WaveSync::sync();
      fft_forward<SC, 1, WaveSync>(v, area, lay, tw, t);
      axis_phase<T, SC, 1>(v, fz, csign, t);
      fft_inverse<SC, 1, WaveSync>(v, area, lay, tw, t);
      const auto rs = rsrc(out + wv * npts, (uint32_t)npts);
#pragma unroll
      for (int q = 0; q < E; ++q)
        st(rs, own_idx<N, E, SC::RF>(t, q) * plane + off0 + col, v[0][q]);
    }
  }
}

// ---------------------------------------------------------------- y-pass
// One surface `psi_s` [N^3]; block (bx, z) owns columns bx*C .. bx*C+C-1 of
// plane z; fy = the y factor; CPOL = cache-policy bits of the loads.
template <typename T, class SC, int C, int CPOL = 0>
__device__ __forceinline__ void ypass_body(cx<T>* __restrict__ psi_s,
                                           const cx<T>* __restrict__ tw,
                                           const cx<T>* __restrict__ fy, int conj, cx<T>* lds,
                                           int bx, int z, int lane = (int)threadIdx.x,
                                           const cx<T>* src_s = nullptr) {
  constexpr int N = SC::N, E = SC::E;
  const int col = lane % C, t = lane / C;
  const int x = bx * C + col;
  constexpr int64_t plane = (int64_t)N * N;
  const auto base = rsrc(psi_s + z * plane, (uint32_t)plane);
  const auto bin = rsrc((src_s ? src_s : psi_s) + z * plane, (uint32_t)plane);
  const LayStrided lay{col, 0, C};
  cx<T>* const tws = lds + C * N;  // staged twiddles and y factor
  stage_blocks<T, N, 2>(tws, {tw, fy}, lane, C * SC::TPC);
  cx<T> v[1][E];
#pragma unroll
  for (int q = 0; q < E; ++q)
    v[0][q] = ld<T, CPOL>(bin, own_idx<N, E, SC::RF>(t, q) * N + x);
  fft_forward<SC, 1>(v, lds, lay, tws, t);
  axis_phase<T, SC, 1>(v, tws + axis_block<T, N>(), conj ? (T)-1 : (T)1, t);
  fft_inverse<SC, 1>(v, lds, lay, tws, t);
#pragma unroll
  for (int q = 0; q < E; ++q) st(base, own_idx<N, E, SC::RF>(t, q) * N + x, v[0][q]);
}

// ---------------------------------------------------------------- x-pass
// One surface `psi_s`; block (bx, z) owns rows bx*ROWS .. bx*ROWS+ROWS-1 of
// plane z; fx = the x factor.
template <typename T, class SC, int ROWS>
__device__ __forceinline__ void xpass_body(cx<T>* __restrict__ psi_s,
                                           const cx<T>* __restrict__ tw,
                                           const cx<T>* __restrict__ fx, int conj, cx<T>* lds,
                                           int bx, int z, int lane = (int)threadIdx.x,
                                           const cx<T>* src_s = nullptr) {
  constexpr int N = SC::N, E = SC::E, TPC = SC::TPC;
  const int t = lane % TPC, row = lane / TPC;
  const int y = bx * ROWS + row;
  constexpr int64_t plane = (int64_t)N * N;
  const auto base = rsrc(psi_s + z * plane, (uint32_t)plane);
  const auto bin = rsrc((src_s ? src_s : psi_s) + z * plane, (uint32_t)plane);
  const uint32_t yo = (uint32_t)y * N;
  const LayPadded lay{row * (N + N / 16), 0};
  cx<T>* const tws = lds + ROWS * (N + N / 16);  // staged twiddles and x factor
  stage_blocks<T, N, 2>(tws, {tw, fx}, lane, ROWS * TPC);
  cx<T> v[1][E];
#pragma unroll
  for (int q = 0; q < E; ++q) v[0][q] = ld<T>(bin, own_idx<N, E, SC::RF>(t, q) + yo);
  fft_forward<SC, 1>(v, lds, lay, tws, t);
  axis_phase<T, SC, 1>(v, tws + axis_block<T, N>(), conj ? (T)-1 : (T)1, t);
  fft_inverse<SC, 1>(v, lds, lay, tws, t);
#pragma unroll
  for (int q = 0; q < E; ++q) st(base, own_idx<N, E, SC::RF>(t, q) + yo, v[0][q]);
}

// ---------------------------------------------------------------- xy plane
// The y- and x-passes of one kinetic action fused for grids whose whole xy
// plane fits in LDS: block = one plane z of one surface, N x TPC threads.
// The y round trip runs in the column layout (a wave holds 64 / TPC columns),
// one LDS transpose moves the plane to the row layout (lane -> t = lane % TPC,
// y = lane / TPC), where the x round trip runs and the rows are stored.  Every
// pencil sees the same stages, twiddles and factors as in the separate passes,
// so the values are identical.
// A single state has fewer planes than there are compute units (32^3 x 3: 96
// of 2 waves), so the pass is the time of one plane: a chain of loads, LDS
// round trips and butterflies.  A wave owns whole pencils in both layouts, so
// that only the transpose needs barriers; the tables are loaded before the
// data and staged while these arrive; twiddles are held in registers (64^3:
// 12.5 -> 11.9 us, 48^3: 8.1 -> 7.7 us against reads between the stages); 48
// points take two stages, 12 x 4, not 4 x 4 x 3.  us a pass (FP64), before ->
// now: 32^3 x 3: 4.8 -> 4.5, 48^3 x 2: 10.4 -> 7.7, 64^3 x 3: 12.7 -> 11.7 (of
// which a copy of the same data takes 2.7, 4.6 and 7.4), all behind the z tile.
// A trace shows less behind a slower z-pass, whose writes are out by its end:
// 64^3 x 3, z + plane: 13.2 + 10.9 with neither, 10.6 + 12.7 with the z tile, 10.6 +
// 11.7 with both; ten TJ-4 steps 798, 782 and 736 us.
template <typename T, class SC>
constexpr size_t plane_lds_elems() {
  return (size_t)SC::N * (SC::N + SC::N / 16) + 4 * axis_block<T, SC::N>();
}
template <typename T, class SC>
constexpr bool plane_fits() {
  return plane_lds_elems<T, SC>() * sizeof(cx<T>) <= 160 * 1024 && SC::N * SC::TPC <= 1024;
}

// Workgroups of up to 512 threads take the columns by waves, with the twiddles
// in registers.  Of 1024 threads (128^3 FP32) each has 128 registers, which do
// not hold them (34 spilled), and a wave's 8 columns would be 64-byte pieces: 64
// neighbouring columns a wave there, block barriers between the columns' stages
// and twiddles read from LDS (S = 3, five TJ-4 steps: 1425 -> 1325 us).
template <class SC>
constexpr bool plane_waves() {
  return SC::N * SC::TPC <= 512;
}
// One pencil's transforms with the twiddles in registers (REGS) or in LDS.
template <typename T, class SC, bool REGS>
struct PlaneTw {
  TwRegs<T, SC> r;
  __device__ __forceinline__ void load(const cx<T>* tw, int t) { r.load(tw, t); }
  template <class Sync, class Lay>
  __device__ __forceinline__ void forward(cx<T> (*v)[SC::E], cx<T>* lds, const Lay& lay, int t) {
    fft_forward<SC, Sync>(v, lds, lay, r, t);
  }
  template <class Sync, class Lay>
  __device__ __forceinline__ void inverse(cx<T> (*v)[SC::E], cx<T>* lds, const Lay& lay, int t) {
    fft_inverse<SC, Sync>(v, lds, lay, r, t);
  }
};
template <typename T, class SC>
struct PlaneTw<T, SC, false> {
  const cx<T>* tw;
  __device__ __forceinline__ void load(const cx<T>* src, int) { tw = src; }
  template <class Sync, class Lay>
  __device__ __forceinline__ void forward(cx<T> (*v)[SC::E], cx<T>* lds, const Lay& lay, int t) {
    fft_forward<SC, 1, Sync>(v, lds, lay, tw, t);
  }
  template <class Sync, class Lay>
  __device__ __forceinline__ void inverse(cx<T> (*v)[SC::E], cx<T>* lds, const Lay& lay, int t) {
    fft_inverse<SC, 1, Sync>(v, lds, lay, tw, t);
  }
};

// `kin` = the three per-axis factors [f_z | f_y | f_x] of one kinetic set.
template <typename T, class SC>
__device__ __forceinline__ void plane_body(cx<T>* __restrict__ psi_s,
                                           const cx<T>* __restrict__ tw,
                                           const cx<T>* __restrict__ kin, int conj, cx<T>* lds,
                                           int z) {
  constexpr int N = SC::N, E = SC::E, TPC = SC::TPC;
  constexpr int P = N + N / 16;  // padded row stride in LDS
  constexpr bool WAVES = plane_waves<SC>();
  using ColSync = std::conditional_t<WAVES, WaveSync, BlockSync>;
  const int lane = threadIdx.x;
  // column layout: with WAVES a wave holds 64 / TPC whole columns
  constexpr int CW = 64 / TPC;
  const int col = WAVES ? lane / 64 * CW + lane % CW : lane % N;
  const int tc = WAVES ? lane % 64 / CW : lane / N;
  const int tr = lane % TPC, row = lane / TPC;  // row layout
  constexpr int64_t plane = (int64_t)N * N;
  const auto base = rsrc(psi_s + z * plane, (uint32_t)plane);
  constexpr int AS = axis_block<T, N>();  // axis stride of the twiddle and factor blocks
  // staged [twiddles y | twiddles x | f_y | f_x] after the plane
  cx<T>* const twy = lds + N * P;
  cx<T>* const twx = twy + AS;
  // the two axes' twiddles and factors, one 16-byte entry a thread
  static_assert(4 * N <= N * TPC, "one entry a thread");
  const sop_u32x4* const p16 =
      reinterpret_cast<const sop_u32x4*>(lane < 2 * N ? tw : kin - 2 * AS) + N + lane;
  sop_u32x4 entry = {};
  if (lane < 4 * N) entry = *p16;
  cx<T> v[1][E];
#pragma unroll
  for (int q = 0; q < E; ++q) v[0][q] = ld<T>(base, own_idx<N, E, SC::RF>(tc, q) * N + col);
  if (lane < 4 * N) reinterpret_cast<sop_u32x4*>(twy)[lane] = entry;
  const LayStrided lcol{col, 0, N};
  const LayPadded lrow{row * P, 0};
  const T csign = conj ? (T)-1 : (T)1;
  // y round trip (columns); without WAVES the first exchange's barrier orders
  // the staged tables
  if constexpr (WAVES) __syncthreads();
  PlaneTw<T, SC, WAVES> tws;
  tws.load(twy, tc);
  tws.template forward<ColSync>(v, lds, lcol, tc);
  axis_phase<T, SC, 1>(v, twy + 2 * AS, csign, tc);
  tws.template inverse<ColSync>(v, lds, lcol, tc);
  if constexpr (WAVES) __syncthreads();
  // columns -> rows
#pragma unroll
  for (int q = 0; q < E; ++q) lds[own_idx<N, E, SC::RF>(tc, q) * P + col] = v[0][q];
  tws.load(twx, tr);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < E; ++q) v[0][q] = lds[row * P + own_idx<N, E, SC::RF>(tr, q)];
  WaveSync::sync();
  // x round trip (rows, whole ones in a wave)
  tws.template forward<WaveSync>(v, lds, lrow, tr);
  axis_phase<T, SC, 1>(v, twy + 3 * AS, csign, tr);
  tws.template inverse<WaveSync>(v, lds, lrow, tr);
#pragma unroll
  for (int q = 0; q < E; ++q) st(base, row * N + own_idx<N, E, SC::RF>(tr, q), v[0][q]);
}

}  // namespace sop
