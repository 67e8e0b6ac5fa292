// body_1d.hpp -- the composed time step of a one-dimensional wavepacket as a
// device function run by one workgroup.
//
// The S-surface state stays in registers (radix-R_first ownership) for all
// nsteps x (N_A + N_B) actions of the pruned sequence (Sec. "Pruning
// splitting coefficients"); only the FFT stage exchanges touch LDS, and HBM
// sees psi at entry and exit.  A potential action is the S x S matvec with
// the stored table exp(-i a dt V(x)/hbar) of its unique coefficient
// (Eq. range_index_unq); a kinetic action is forward FFT -> phase (with 1/N
// folded in) -> inverse FFT (Sec. "Dynamic Fourier method").  conj = 1
// conjugates every table, which is U(-dt).  At a step boundary inside the
// call the two adjoining actions of one kind run as one (DevView::mid).
#pragma once

#include "fft_core.hpp"
#include "internal.hpp"

namespace sop {

namespace s1d {
// schedules: (N, E, forward radices, inverse radices = reversed, first, last).
// Eight values per thread and surface keep a two-surface FP64 state plus a
// radix-8 butterfly in about 128 VGPRs.
using S16 = Sched<16, 4, RList<4, 4>, RList<4, 4>, 4, 4>;
using S32 = Sched<32, 8, RList<8, 4>, RList<4, 8>, 8, 4>;
using S64 = Sched<64, 8, RList<8, 8>, RList<8, 8>, 8, 8>;
using S128 = Sched<128, 8, RList<8, 4, 4>, RList<4, 4, 8>, 8, 4>;
using S256 = Sched<256, 8, RList<8, 8, 4>, RList<4, 8, 8>, 8, 4>;
using S512 = Sched<512, 8, RList<8, 8, 8>, RList<8, 8, 8>, 8, 8>;
using S1024 = Sched<1024, 8, RList<8, 4, 4, 8>, RList<8, 4, 4, 8>, 8, 8>;
using S2048 = Sched<2048, 8, RList<8, 8, 4, 8>, RList<8, 4, 8, 8>, 8, 8>;
using S4096 = Sched<4096, 8, RList<8, 8, 8, 8>, RList<8, 8, 8, 8>, 8, 8>;
using S8192 = Sched<8192, 8, RList<8, 8, 8, 8, 2>, RList<2, 8, 8, 8, 8>, 8, 2>;
}  // namespace s1d

// LDS slots of one pencil: one padding slot per 16 elements.
template <class SC>
constexpr int lds_pencil() {
  return SC::N + SC::N / 16;
}

// GUARD: pass the thread index through opaque() for every transform and
// action, so that twiddles and addresses are recomputed instead of being
// held for the whole run.  Measured per step on gfx950 (two surfaces, FP64):
// N = 8192 55 us guarded vs 141 us held (spilled); 512 and 2048 slightly
// faster guarded; 1024 slightly faster without.  At N = 4096 the held FP64
// kernel spills (256 VGPRs and 400 bytes of scratch a lane) and the guarded
// one does not (178 VGPRs): 17.8 against 20.8 us a substep; in FP32 nothing
// spills and holding is faster (12.3 against 14.5 us).
template <typename T>
constexpr bool guard_default(int n) {
  return n == 512 || n == 2048 || n >= 8192 || (n == 4096 && sizeof(T) == 8);
}
template <bool GUARD>
__device__ __forceinline__ int guard(int t) {
  if constexpr (GUARD) return opaque(t);
  else return t;
}

// Walk over the actions of a run of NT threads.  Plain: the program (nact
// actions) once per step.  With merged step boundaries (mid), `prog` holds the
// program with the merged action before its last one, a_1 .. a_{n-1} mid a_n:
// every step but the first starts at a_2 and every step but the last ends with
// mid.  The lanes of each wave hold a piece of the program, one entry each,
// and the current entry is read from its lane: a load of every entry from
// memory would stand at the head of each action's chain.
template <int NT>
struct Walk {
  static constexpr int CH = NT < 64 ? NT : 64;  // entries of a piece
  const int* prog;
  int len, again, end, last;
  int pos = 0, base = 0, piece;
  int64_t left;  // actions to run
  __device__ __forceinline__ Walk(const int* prog_, int nact, int64_t nsteps, int mid) {
    const int body = mid ? nact - 1 : nact;  // actions a further step adds
    prog = prog_;
    len = mid ? nact + 1 : nact;
    end = nact;
    again = mid ? 1 : 0;
    last = len - 1;
    left = nsteps > 0 ? nsteps * body + again : 0;
    fetch();
  }
  __device__ __forceinline__ void fetch() {
    const int i = base + (int)threadIdx.x % CH;
    piece = prog[i < len ? i : len - 1];
  }
  __device__ __forceinline__ int code() const {
    return __builtin_amdgcn_readlane(piece, pos - base);
  }
  __device__ __forceinline__ void next() {
    --left;
    ++pos;
    if (pos == end) pos = again;
    if (left == 1) pos = last;
    if (pos < base || pos >= base + CH) {
      base = pos - pos % CH;
      fetch();
    }
  }
};

// Whether the program is held by the lanes (Walk, one loop over the actions) or
// read from memory by nested loops over pieces and steps, in the single-plan
// kernels.  A workgroup of N / 8 threads holds a piece of N / 8 entries: on long
// programs the grids of up to 128 points spent their time refilling it (us of 1500 substeps of
// triple-jump-8, held / nested: FP64 16 x 1 1480 / 1060, 64 x 2 3890 / 3650, 128 x 1
// 3290 / 3040; FP32 128 x 1 3760 / 3050).  From 512 points on the nested loops
// lose (FP32 512 x 1 4210 / 4850; FP64 8192 x 1, 500 substeps, 12490 / 13340), and on
// four short grids the compiler holds more of the twiddles in the one loop (156
// against 136 registers at FP64 64 x 1): FP64 32 x 1 2090 / 2450, 64 x 1 2260 / 2500,
// 256 x 1 3350 / 3920; FP32 64 x 2 4540 / 5310.  Two FP64 surfaces of 8192 points
// have registers for neither (500 substeps held 25300, nested 23300, without
// merged boundaries 22300: merge_potential).
template <typename T>
constexpr bool walk_held(int n, int S) {
  if (sizeof(T) == 4) return n >= 512 || (n == 64 && S == 2);
  if (n < 512) return S == 1 && (n == 32 || n == 64 || n == 256);
  return merge_potential(n, S, true);
}

// One action of the program (code) on the state held in registers.
template <typename T, class SC, int S, int PL, bool GUARD>
__device__ __forceinline__ void action(cx<T> (&v)[S][SC::E], int code, const cx<T>* vexp,
                                       const cx<T>* kin, const cx<T>* tw, T csign, cx<T>* lds,
                                       int t0) {
  constexpr int N = SC::N, E = SC::E, NE = S * (S + 1) / 2;
  // the tables of a length with a body on waves are stored in that body's order
  constexpr int W = wave_body(N, S);
  auto place_x = [](int x) { return W ? wave_order_x(W ? W : 1, x) : x; };
  auto place_k = [](int k) { return W ? wave_order_k(W ? W : 1, k) : k; };
  const LayPadded lay{0, lds_pencil<SC>()};
  const int idx = code & 0xffff;
  const int t = guard<GUARD>(t0);
  if ((code >> 16) == OP_V) {
    // table entries are (rounded, residue) pairs in FP32
    const cx<T>* U = vexp + (size_t)idx * NE * N * Split<T>::rep;
#pragma unroll
    for (int q = 0; q < E; ++q) {
      const int x = own_idx<N, E, SC::RF>(t, q);
      Fac<T> u[NE];
#pragma unroll
      for (int e = 0; e < NE; ++e) u[e] = load_fac(U, e * N + place_x(x), csign);
      cx<T> w[S];
#pragma unroll
      for (int s = 0; s < S; ++s) w[s] = v[s][q];
      apply_u_fac<T, S>(w, u);
#pragma unroll
      for (int s = 0; s < S; ++s) v[s][q] = w[s];
    }
  } else {
    if constexpr (PL == S && S == 2) {
      fft_forward_pair2<SC>(v, lds, lay, tw, guard<GUARD>(t0));
    } else if constexpr (PL == S) {
      fft_forward<SC, S>(v, lds, lay, tw, guard<GUARD>(t0));
    } else if constexpr (S == 2) {
      fft_forward_pair<SC>(v, lds, lay, tw, guard<GUARD>(t0));
    } else {
#pragma unroll
      for (int s = 0; s < S; ++s) fft_forward<SC, 1>(v + s, lds, lay, tw, guard<GUARD>(t0));
    }
    const cx<T>* F = kin + (size_t)idx * N * Split<T>::rep;
#pragma unroll
    for (int q = 0; q < E; ++q) {
      const Fac<T> f = load_fac(F, place_k(own_idx<N, E, SC::RL>(t, q)), csign);
#pragma unroll
      for (int s = 0; s < S; ++s) v[s][q] = fmul(v[s][q], f);
    }
    if constexpr (PL == S && S == 2) {
      fft_inverse_pair2<SC>(v, lds, lay, tw, guard<GUARD>(t0));
    } else if constexpr (PL == S) {
      fft_inverse<SC, S>(v, lds, lay, tw, guard<GUARD>(t0));
    } else if constexpr (S == 2) {
      fft_inverse_pair<SC>(v, lds, lay, tw, guard<GUARD>(t0));
    } else {
#pragma unroll
      for (int s = 0; s < S; ++s) fft_inverse<SC, 1>(v + s, lds, lay, tw, guard<GUARD>(t0));
    }
  }
}

// PL = pencils exchanged through LDS at once (S, or 1 when S pencils do not
// fit).  `lds` holds PL padded pencils.  With one pencil of buffer and two
// surfaces the two transforms run interleaved (fft_forward_pair).
// MERGE: the run may have merged step boundaries (mid).  HELD: the walk.
template <typename T, class SC, int S, int PL,
          bool GUARD = guard_default<T>(SC::N), bool MERGE = true,
          bool HELD = walk_held<T>(SC::N, S)>
__device__ __forceinline__ void run_1d(cx<T>* __restrict__ psi, const cx<T>* __restrict__ vexp,
                                       const cx<T>* __restrict__ kin,
                                       const cx<T>* __restrict__ tw,
                                       const int* __restrict__ prog, int nact, int64_t nsteps,
                                       int conj, int mid, cx<T>* lds) {
  const int t0 = threadIdx.x;
  constexpr int N = SC::N, E = SC::E;
  const T csign = conj ? (T)-1 : (T)1;
  cx<T> v[S][E];
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int q = 0; q < E; ++q) v[s][q] = psi[s * N + own_idx<N, E, SC::RF>(t0, q)];

  if constexpr (HELD) {
    for (Walk<SC::TPC> w(prog, nact, nsteps, mid); w.left > 0; w.next())
      action<T, SC, S, PL, GUARD>(v, w.code(), vexp, kin, tw, csign, lds, t0);
  } else {
    // pieces of a run with merged boundaries: a_1 .. a_{n-1} mid once, a_2 ..
    // a_{n-1} mid nsteps - 2 times, a_2 .. a_n once (the plain program precedes
    // the list with mid)
    const bool pieces = MERGE && mid && nsteps > 1;
    const int* list = MERGE && mid && !pieces ? prog - nact : prog;
    int len = nact;
    int64_t reps = pieces ? 1 : nsteps;
    for (int p = pieces ? 0 : 2; p < 3; ++p) {
      for (int64_t step = 0; step < reps; ++step)
        for (int a = 0; a < len; ++a)
          action<T, SC, S, PL, GUARD>(v, list[a], vexp, kin, tw, csign, lds, t0);
      if constexpr (!MERGE) break;
      list = p == 0 ? prog + 1 : prog - nact + 1;
      len = nact - 1;
      reps = p == 0 ? nsteps - 2 : 1;
    }
  }
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int q = 0; q < E; ++q) psi[s * N + own_idx<N, E, SC::RF>(t0, q)] = v[s][q];
}

}  // namespace sop
