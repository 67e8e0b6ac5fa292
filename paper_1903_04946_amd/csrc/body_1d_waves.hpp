// body_1d_waves.hpp -- the composed time step of a two-surface wavepacket of
// N = 256 W points on W waves (W = 1, 2, 4, 8).
//
// Same step as run_1d (Sec. "Dynamic Fourier method"; the pruned action
// sequence of Sec. "Pruning splitting coefficients"), with the work laid out
// so that a lane holds one surface only, the exchanges of a transform stay
// inside one wave but for one, and one of them needs no LDS:
//
// * 64 W threads hold 8 values each; lane bit 3 selects the surface, so lanes
//   l and l ^ 8 hold the two surfaces at the same points.
// * The DFT of length N is the mixed-radix Cooley-Tukey factorisation
//   8 x 8 x 4 x W written as nested four-step transforms:
//       x = (N/8) x1 + (N/64) y1 + W z1 + z2,
//       k = k1 + 8 k1' + 64 k1'' + 256 k2'',
//   radix-8 DFT over x1, twiddle w_N^(x2 k1) (x2 = x mod N/8), radix-8 over y1,
//   twiddle w_(N/8)^(y2 k1') (y2 = x mod N/64), radix-4 over z1, twiddle
//   w_(4W)^(z2 k1''), radix-W over z2.  The inverse runs the same steps in
//   reverse order with conjugate roots (the unnormalised inverse DFT; the
//   1/N sits in the kinetic factors).
// * Ownership (wave w; lane l = 16 h + 8 s + g, h < 4, g < 8; register r):
//       position side   x = (N/8) r + (N/64) g + W h + w    (g = y1, h = z1, w = z2)
//       after stage 1   g = y1, h = z1, register k1
//       after stage 2   g = k1, h = z1, register k1'
//       after stage 3   g = k1, h = c, register (k1'' = r % 4, c2 = r / 4),
//                       where k1' = c + 4 c2; wave z2
//       frequency side  register bits (k1'', c2) low ones first: log2 W of them in
//                       the wave, k2'' in the register's low bits, the rest above
//                       (wave_order_k)
// * Exchange A (stage 1 -> 2) swaps the three register bits with the lane bits
//   of g, through the wave's own LDS region: a wavefront's LDS operations
//   complete in issue order, so it needs a compiler fence, no barrier.
//   Exchange B (2 -> 3) swaps two register bits with lane bits 4 and 5, which
//   v_permlane16_swap and v_permlane32_swap do in registers.  Exchange C
//   (3 -> 4, W > 1) swaps register and wave bits through a shared region
//   behind one barrier.  The inverse transform's exchange C writes exactly
//   the slots the same thread read in the forward one and reads the slots it
//   wrote there, so the one buffer needs no second barrier: a thread only
//   ever overwrites slots it has already read.
// * The potential action takes the other surface's value at each point from
//   lane l ^ 8 (a DPP row rotation by 8) and forms its own row of the 2 x 2
//   product; its table entries are requested before the inverse transform of
//   the kinetic action before it.
//
// What bounds it: one wave per SIMD (two at W = 8) runs one chain of
// arithmetic (W = 4: 731 VALU instructions a substep in FP64, 1.2 us at 4 cycles
// each) and LDS round trips (0.2 us of the CU's LDS rate an exchange plus its
// latency), little of which overlaps.
#pragma once

#include "body_1d.hpp"

namespace sop {
namespace wv {

template <int W>
struct Dim {
  static constexpr int N = 256 * W;
  static constexpr int threads = 64 * W;
  static constexpr int kRow = 65;           // slots per k1 row of a wave region (64 lanes + 1)
  static constexpr int kWave = 8 * kRow;    // slots per wave region
  static constexpr int kCross = W * kWave;  // first slot of the shared region
  static constexpr int kSlots = kCross + (W > 1 ? 2 * N : 0);
};
template <typename T, int W>
constexpr size_t lds_bytes() {
  return (size_t)Dim<W>::kSlots * sizeof(cx<T>);
}

// Compiler fence for LDS traffic within one wave (the hardware already keeps
// a wave's LDS operations in order).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}
// Workgroup barrier ordering LDS only: global loads in flight (kinetic
// factors, table entries) stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Index maps of one thread.
template <int W>
struct Map {
  using D = Dim<W>;
  int w, l, g, h, s;
  int wa;  // LDS region of this wave
  __device__ __forceinline__ Map(int tid) {
    l = tid & 63;
    w = W > 1 ? tid >> 6 : 0;
    g = l & 7;
    s = (l >> 3) & 1;
    h = l >> 4;
    wa = w * D::kWave;
  }
  __device__ __forceinline__ int pos(int r) const {
    return (D::N / 8) * r + (D::N / 64) * g + W * h + w;
  }
  // table place of register 0's point and frequency (32 more a register)
  __device__ __forceinline__ int place() const { return 256 * w + 8 * h + g; }
  // A: element k1 of lane (h, s, y1) at row k1, column l.  One side's accesses
  // are contiguous; on the other the eight lanes g of a group go to eight rows,
  // whose length of 64 + 1 slots puts them, and the groups a 16-byte read takes
  // together, on distinct banks (no conflicts counted; rows of 33 per surface
  // had 256 conflict cycles a substep at W = 4).
  __device__ __forceinline__ int a_t(int r) const { return wa + r * D::kRow + l; }
  __device__ __forceinline__ int a_f(int r) const { return wa + g * D::kRow + l - g + r; }
  // C: the exchanged register bits (low ones first) and the wave, then the
  // other register bits, then the lane
  __device__ __forceinline__ int c_t(int r) const {
    constexpr int K = 8 / W;  // register values that stay
    return D::kCross + (((r % W) * W + w) * K + r / W) * 64 + l;
  }
  __device__ __forceinline__ int c_f(int r) const {
    constexpr int K = 8 / W;
    return D::kCross + ((w * W + r % W) * K + r / W) * 64 + l;
  }
};

// Exchange inside the wave: write through `wr`, read through `rd`.
template <typename T, class WR, class RD>
__device__ __forceinline__ void xwave(cx<T> (&v)[8], cx<T>* lds, WR wr, RD rd) {
#pragma unroll
  for (int r = 0; r < 8; ++r) lds[wr(r)] = v[r];
  wave_sync();
#pragma unroll
  for (int r = 0; r < 8; ++r) v[r] = lds[rd(r)];
  wave_sync();
}
// Exchange across the waves (one barrier; see the header for the second).
template <typename T, class WR, class RD>
__device__ __forceinline__ void xcross(cx<T> (&v)[8], cx<T>* lds, WR wr, RD rd) {
#pragma unroll
  for (int r = 0; r < 8; ++r) lds[wr(r)] = v[r];
  lds_barrier();
#pragma unroll
  for (int r = 0; r < 8; ++r) v[r] = lds[rd(r)];
  wave_sync();
}

template <typename T>
struct Words {
  static constexpr int n = (int)(sizeof(cx<T>) / 4);
  uint32_t u[n];
};
// Swaps the register bit that tells `a` (0) from `b` (1) with lane bit 5 or 4.
template <int BIT, typename T>
__device__ __forceinline__ void swap_bit(cx<T>& a, cx<T>& b) {
  Words<T> p = __builtin_bit_cast(Words<T>, a), q = __builtin_bit_cast(Words<T>, b);
#pragma unroll
  for (int i = 0; i < Words<T>::n; ++i) {
    const auto x = BIT == 5 ? __builtin_amdgcn_permlane32_swap(p.u[i], q.u[i], false, false)
                            : __builtin_amdgcn_permlane16_swap(p.u[i], q.u[i], false, false);
    p.u[i] = x[0];
    q.u[i] = x[1];
  }
  a = __builtin_bit_cast(cx<T>, p);
  b = __builtin_bit_cast(cx<T>, q);
}
// Exchange B, its own inverse: register bits 0, 1 with lane bits 4, 5.
template <typename T>
__device__ __forceinline__ void xlanes(cx<T> (&v)[8]) {
#pragma unroll
  for (int c = 0; c < 8; c += 4) {
    swap_bit<4>(v[c], v[c + 1]);
    swap_bit<4>(v[c + 2], v[c + 3]);
    swap_bit<5>(v[c], v[c + 2]);
    swap_bit<5>(v[c + 1], v[c + 3]);
  }
}
// The value of lane l ^ 8 (a rotation by 8 of each row of 16 lanes).
template <typename T>
__device__ __forceinline__ cx<T> other_surface(cx<T> a) {
  Words<T> p = __builtin_bit_cast(Words<T>, a);
#pragma unroll
  for (int i = 0; i < Words<T>::n; ++i)
    p.u[i] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)p.u[i], 0x128, 0xf, 0xf, true);
  return __builtin_bit_cast(cx<T>, p);
}

// a * F, or a * conj(F) when C
template <bool C, typename T>
__device__ __forceinline__ cx<T> fmul_c(cx<T> a, const Fac<T>& F) {
  if constexpr (!C) {
    return fmul(a, F);
  } else {
    Fac<T> G = F;
    G.w.im = -G.w.im;
    if constexpr (std::is_same<T, float>::value) G.lo.im = -G.lo.im;
    return fmul(a, G);
  }
}

// Twiddles of the inner steps, fixed per thread for the whole run.
template <typename T, int W>
struct Tw {
  Fac<T> t1[7], t2[7], t3[3];
  __device__ __forceinline__ void load(const cx<T>* __restrict__ tw, const Map<W>& m) {
    const int y2 = W * m.h + m.w;                // x mod N/64 after stage 1
    const int x2 = Dim<W>::N / 64 * m.g + y2;    // x mod N/8 on the position side
#pragma unroll
    for (int j = 1; j < 8; ++j) {
      t1[j - 1] = load_fac(tw, x2 * j, (T)1);        // w_N^(x2 k1)
      t2[j - 1] = load_fac(tw, 8 * y2 * j, (T)1);    // w_(N/8)^(y2 k1')
    }
    if constexpr (W > 1) {
#pragma unroll
      for (int j = 1; j < 4; ++j) t3[j - 1] = load_fac(tw, 64 * m.w * j, (T)1);  // w_(4W)^(z2 k1'')
    }
  }
};

// radix-W DFTs over the low register bits
template <int W, bool INV, typename T>
__device__ __forceinline__ void dft_waves(cx<T> (&v)[8]) {
  if constexpr (W > 1) {
#pragma unroll
    for (int r = 0; r < 8; r += W) dft<W, INV>(v + r);
  }
}

template <typename T, int W>
__device__ __forceinline__ void forward(cx<T> (&v)[8], cx<T>* lds, const Map<W>& m,
                                        const Tw<T, W>& tw) {
  dft<8, false>(v);
#pragma unroll
  for (int r = 1; r < 8; ++r) v[r] = fmul(v[r], tw.t1[r - 1]);
  xwave(v, lds, [&](int r) { return m.a_t(r); }, [&](int r) { return m.a_f(r); });
  dft<8, false>(v);
#pragma unroll
  for (int r = 1; r < 8; ++r) v[r] = fmul(v[r], tw.t2[r - 1]);
  xlanes(v);
  dft<4, false>(v);
  dft<4, false>(v + 4);
  if constexpr (W > 1) {
#pragma unroll
    for (int r = 1; r < 8; ++r)
      if (r & 3) v[r] = fmul(v[r], tw.t3[(r & 3) - 1]);
    xcross(v, lds, [&](int r) { return m.c_t(r); }, [&](int r) { return m.c_f(r); });
    dft_waves<W, false>(v);
  }
}

template <typename T, int W>
__device__ __forceinline__ void inverse(cx<T> (&v)[8], cx<T>* lds, const Map<W>& m,
                                        const Tw<T, W>& tw) {
  if constexpr (W > 1) {
    dft_waves<W, true>(v);
    xcross(v, lds, [&](int r) { return m.c_f(r); }, [&](int r) { return m.c_t(r); });
#pragma unroll
    for (int r = 1; r < 8; ++r)
      if (r & 3) v[r] = fmul_c<true>(v[r], tw.t3[(r & 3) - 1]);
  }
  dft<4, true>(v);
  dft<4, true>(v + 4);
  xlanes(v);
#pragma unroll
  for (int r = 1; r < 8; ++r) v[r] = fmul_c<true>(v[r], tw.t2[r - 1]);
  dft<8, true>(v);
  xwave(v, lds, [&](int r) { return m.a_f(r); }, [&](int r) { return m.a_t(r); });
#pragma unroll
  for (int r = 1; r < 8; ++r) v[r] = fmul_c<true>(v[r], tw.t1[r - 1]);
  dft<8, true>(v);
}

// own * U_ss + other * U_01 (conjugated factors when C): one row of the 2 x 2
// product.  In FP32 in FP64 on rounded + residue, rounded once (as
// apply_u_fac).
template <bool C, typename T>
__device__ __forceinline__ cx<T> row(cx<T> own, cx<T> oth, const Fac<T>& us, const Fac<T>& uo) {
  if constexpr (std::is_same<T, float>::value) {
    const double sg = C ? -1.0 : 1.0;
    const cx<double> a = {(double)us.w.re + (double)us.lo.re,
                          sg * ((double)us.w.im + (double)us.lo.im)};
    const cx<double> b = {(double)uo.w.re + (double)uo.lo.re,
                          sg * ((double)uo.w.im + (double)uo.lo.im)};
    const cx<double> r = cadd(cmul(a, cx<double>{(double)own.re, (double)own.im}),
                              cmul(b, cx<double>{(double)oth.re, (double)oth.im}));
    return {(float)r.re, (float)r.im};
  } else {
    return cadd(fmul_c<C>(own, us), fmul_c<C>(oth, uo));
  }
}

// The action loop on a state held in registers.  CONJ applies conj(U) and
// conj(F), which is U(-dt): a compile-time flag, so that the sign folds into
// the products where a factor is used and does not pull its load forward.
// Potential and kinetic actions alternate: one turn of the loop is a
// potential action, if one is next, and the kinetic action after it.
template <typename T, int W, bool CONJ>
__device__ __forceinline__ void actions(cx<T> (&v)[8], const Map<W>& m, const Tw<T, W>& tws,
                                        const cx<T>* __restrict__ vexp,
                                        const cx<T>* __restrict__ kin,
                                        const int* __restrict__ prog, int nact, int64_t nsteps,
                                        int mid, cx<T>* lds) {
  constexpr int N = Dim<W>::N;
  Walk<Dim<W>::threads> walk(prog, nact, nsteps, mid);
  if (walk.left <= 0) return;
  constexpr int REP = Split<T>::rep;
  constexpr uint32_t EB = REP * sizeof(cx<T>);  // bytes of a table entry
  // One lane offset serves all entries of a kind; the registers' distances are
  // constants and the table's base is scalar.  The tables are in wave order:
  // a load of a wave is two runs of 32 entries (in point order it was 32
  // pieces, which kept the address path busy for 1.3 us a substep at W = 4).
  const uint32_t ofr = (uint32_t)m.place() * EB, oss = ofr + 2 * m.s * N * EB, o01 = ofr + N * EB;
  Fac<T> us[8], uo[8];  // entries U_ss and U_01 of the next potential action
  auto table = [&](int idx) {
    const auto rs = rsrc(vexp + (size_t)idx * 3 * N * REP, 3 * N * REP);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      us[r] = ldfac_at<T>(rs, oss, 32 * r * EB);
      uo[r] = ldfac_at<T>(rs, o01, 32 * r * EB);
    }
  };
  int code = walk.code();
  table((code >> 16) == OP_V ? code & 0xffff : 0);
  while (walk.left > 0) {
    if ((code >> 16) == OP_V) {
#pragma unroll
      for (int r = 0; r < 8; ++r) v[r] = row<CONJ>(v[r], other_surface(v[r]), us[r], uo[r]);
      walk.next();
      if (walk.left == 0) break;
      code = walk.code();
    }
    // the factors are requested before the forward transform
    const auto rf = rsrc(kin + (size_t)(code & 0xffff) * N * REP, N * REP);
    Fac<T> kf[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) kf[r] = ldfac_at<T>(rf, ofr, 32 * r * EB);
    forward(v, lds, m, tws);
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = fmul_c<CONJ>(v[r], kf[r]);
    // The next potential action's entries are requested before the inverse
    // transform, and after the factors are used: loads return in order, and a
    // wait for the factors would be a wait for these too.  Without a branch
    // (table 0 if no potential action follows): behind one the compiler
    // cannot count the loads in flight and waits for all.
    __builtin_amdgcn_sched_barrier(0);
    walk.next();
    code = walk.left > 0 ? walk.code() : 0;
    table((code >> 16) == OP_V ? code & 0xffff : 0);
    inverse(v, lds, m, tws);
  }
}

// One potential action alone (one ends every step of a driven run): no
// twiddles, and points dealt so that neighbouring lanes take neighbouring
// points (w) and table entries (g) in runs of 8, where the loop's ownership
// reads and writes the state in 16-byte pieces (2048 points FP64: 7.9 -> 4.9 us,
// 512: 3.3 -> 1.9).  A kernel of its own: as a branch of run it cost 256 points
// 0.8% of every run.
template <typename T, int W>
__device__ __forceinline__ void potential(cx<T>* __restrict__ psi, const cx<T>* __restrict__ vexp,
                                          int idx, int conj) {
  constexpr int N = Dim<W>::N, P = N / Dim<W>::threads;
  const cx<T>* const U = vexp + (size_t)idx * 3 * N * Split<T>::rep;
  const T csign = conj ? (T)-1 : (T)1;
  cx<T> v[P][2];
  Fac<T> u[P][3];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int i = (int)threadIdx.x + p * Dim<W>::threads;
    const int w = i % W, g = i / W % 8, h = i / (8 * W) % 4, r = i / (32 * W);
    const int x = 32 * W * r + 4 * W * g + W * h + w;
#pragma unroll
    for (int s = 0; s < 2; ++s) v[p][s] = psi[s * N + x];
#pragma unroll
    for (int e = 0; e < 3; ++e) u[p][e] = load_fac(U, e * N + wave_order_x(W, x), csign);
  }
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int i = (int)threadIdx.x + p * Dim<W>::threads;
    const int w = i % W, g = i / W % 8, h = i / (8 * W) % 4, r = i / (32 * W);
    const int x = 32 * W * r + 4 * W * g + W * h + w;
    psi[x] = row<false>(v[p][0], v[p][1], u[p][0], u[p][1]);
    psi[N + x] = row<false>(v[p][1], v[p][0], u[p][2], u[p][1]);
  }
}

// The composed step (arguments as in run_1d, S = 2, N = 256 W, 64 W threads,
// lds_bytes<T, W>() bytes of LDS).
template <typename T, int W>
__device__ __forceinline__ void run(cx<T>* __restrict__ psi, const cx<T>* __restrict__ vexp,
                                    const cx<T>* __restrict__ kin, const cx<T>* __restrict__ tw,
                                    const int* __restrict__ prog, int nact, int64_t nsteps,
                                    int conj, int mid, cx<T>* lds) {
  const Map<W> m((int)threadIdx.x);
  Tw<T, W> tws;
  tws.load(tw, m);
  cx<T> v[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    v[r] = psi[m.s * Dim<W>::N + m.pos(r)];
    // consumed here, so no load of psi is outstanding inside the action loop
    asm volatile("" : "+v"(v[r].re), "+v"(v[r].im));
  }
  if (conj)
    actions<T, W, true>(v, m, tws, vexp, kin, prog, nact, nsteps, mid, lds);
  else
    actions<T, W, false>(v, m, tws, vexp, kin, prog, nact, nsteps, mid, lds);
#pragma unroll
  for (int r = 0; r < 8; ++r) psi[m.s * Dim<W>::N + m.pos(r)] = v[r];
}

}  // namespace wv
}  // namespace sop
