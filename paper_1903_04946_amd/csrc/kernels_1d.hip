// kernels_1d.hip -- one-dimensional grids: the whole composed time step runs
// inside one persistent workgroup per wavepacket (the step body is run_1d).
#include "body_1d.hpp"
#include "body_1d_waves.hpp"
#include "reduce.hpp"

namespace sop {
namespace {

using namespace s1d;

// PL = pencils exchanged through LDS at once (S, or 1 when S pencils do not fit).
template <typename T, class SC, int S, int PL, bool MERGE = true>
__global__ void __launch_bounds__(SC::TPC)
    k1d_prop_kernel(cx<T>* __restrict__ psi, const cx<T>* __restrict__ vexp,
                    const cx<T>* __restrict__ kin, const cx<T>* __restrict__ tw,
                    const int* __restrict__ prog, int nact, int64_t nsteps, int conj, int mid) {
  extern __shared__ char smem_raw[];
  cx<T>* lds = reinterpret_cast<cx<T>*>(smem_raw);
  psi += (size_t)blockIdx.x * S * SC::N;  // one workgroup per state
  run_1d<T, SC, S, PL, guard_default<T>(SC::N), MERGE>(psi, vexp, kin, tw, prog, nact, nsteps,
                                                       conj, mid, lds);
}

// Two surfaces of 256 W points: the body on W waves.
template <typename T, int W>
__global__ void __launch_bounds__(wv::Dim<W>::threads)
    k1d_waves_kernel(cx<T>* __restrict__ psi, const cx<T>* __restrict__ vexp,
                     const cx<T>* __restrict__ kin, const cx<T>* __restrict__ tw,
                     const int* __restrict__ prog, int nact, int64_t nsteps, int conj, int mid) {
  extern __shared__ char smem_raw[];
  cx<T>* lds = reinterpret_cast<cx<T>*>(smem_raw);
  psi += (size_t)blockIdx.x * 2 * wv::Dim<W>::N;  // one workgroup per state
  wv::run<T, W>(psi, vexp, kin, tw, prog, nact, nsteps, conj, mid, lds);
}

// One potential action (table entry block idx) of two surfaces of 256 W points.
template <typename T, int W>
__global__ void __launch_bounds__(wv::Dim<W>::threads)
    k1d_waves_potential(cx<T>* __restrict__ psi, const cx<T>* __restrict__ vexp, int idx,
                        int conj) {
  wv::potential<T, W>(psi + (size_t)blockIdx.x * 2 * wv::Dim<W>::N, vexp, idx, conj);
}

// Observables of one state in one workgroup: out[0..S) = sum |psi_s|^2,
// out[S] = sum psi^dag V psi, out[S + 1] = ck sum k^2 |F psi|^2 (k signed; FP64
// sums in a fixed order).
template <typename T, class SC, int S>
__global__ void __launch_bounds__(SC::TPC)
    k1d_obs_kernel(const cx<T>* __restrict__ psi, const double* __restrict__ vraw,
                   const cx<T>* __restrict__ tw, double ck, double* __restrict__ out) {
  extern __shared__ char smem_raw[];
  cx<T>* lds = reinterpret_cast<cx<T>*>(smem_raw);
  constexpr int N = SC::N, E = SC::E;
  const int t = threadIdx.x;
  cx<T> v[S][E];
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int q = 0; q < E; ++q) v[s][q] = psi[s * N + own_idx<N, E, SC::RF>(t, q)];
  double acc[S + 2];
#pragma unroll
  for (int k = 0; k < S + 2; ++k) acc[k] = 0.0;
#pragma unroll
  for (int q = 0; q < E; ++q) {
    const int x = own_idx<N, E, SC::RF>(t, q);
    int e = 0;
#pragma unroll
    for (int i = 0; i < S; ++i)
#pragma unroll
      for (int j = i; j < S; ++j) {
        // Re(conj(psi_i) psi_j), counted twice off the diagonal
        const double rr = (double)v[i][q].re * (double)v[j][q].re +
                          (double)v[i][q].im * (double)v[j][q].im;
        if (i == j) acc[i] += rr;
        acc[S] += (i == j ? 1.0 : 2.0) * vraw[(size_t)e * N + x] * rr;
        ++e;
      }
  }
  const LayPadded lay{0, lds_pencil<SC>()};
  double a = 0.0;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    fft_forward<SC, 1>(v + s, lds, lay, tw, t);
#pragma unroll
    for (int q = 0; q < E; ++q) {
      const int k = own_idx<N, E, SC::RL>(t, q);
      const double kk = (double)(k < N / 2 ? k : k - N);
      const double re = (double)v[s][q].re, im = (double)v[s][q].im;
      a = fma(kk * kk, fma(re, re, im * im), a);
    }
  }
  acc[S + 1] = ck * a;
  workgroup_sum<SC::TPC, S + 2>(acc, reinterpret_cast<double*>(smem_raw));
  if (t == 0) {
#pragma unroll
    for (int k = 0; k < S + 2; ++k) out[k] = acc[k];
  }
}

constexpr size_t kMaxLds = 160 * 1024;

// Dynamic LDS past 64 KB has to be allowed per kernel.
hipError_t set_lds(const void* k, size_t bytes) {
  if (bytes <= 64 * 1024) return hipSuccess;
  return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

template <typename T, class SC, int S>
hipError_t launch_prop(const DevView& d, void* psi, int64_t nsteps, int conj, int count) {
  constexpr size_t one = (size_t)lds_pencil<SC>() * sizeof(cx<T>);
  TimedLaunch tl(d, KIND_1D, 2.0 * S * SC::N * sizeof(cx<T>) * count);
  if constexpr (wave_body(SC::N, S) > 0) {
    constexpr int W = wave_body(SC::N, S);
    constexpr size_t bytes = wv::lds_bytes<T, W>();
    if (d.nact == 1 && nsteps == 1 && prog_op(d.hprog[0]) == OP_V) {
      hipLaunchKernelGGL((k1d_waves_potential<T, W>), dim3(count), dim3(wv::Dim<W>::threads), 0,
                         d.stream, (cx<T>*)psi, (const cx<T>*)d.vexp, prog_idx(d.hprog[0]), conj);
      return hipGetLastError();
    }
    auto k = k1d_waves_kernel<T, W>;
    const hipError_t e = set_lds((const void*)k, bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3(count), dim3(wv::Dim<W>::threads), bytes, d.stream, (cx<T>*)psi,
                       (const cx<T>*)d.vexp, (const cx<T>*)d.kin, (const cx<T>*)d.tw[0],
                       d.prog_1d(), d.nact, nsteps, conj, d.merged());
  } else if (one * S <= kMaxLds) {
    auto k = k1d_prop_kernel<T, SC, S, S>;
    const hipError_t e = set_lds((const void*)k, one * S);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3(count), dim3(SC::TPC), one * S, d.stream, (cx<T>*)psi,
                       (const cx<T>*)d.vexp, (const cx<T>*)d.kin, (const cx<T>*)d.tw[0], d.prog_1d(),
                       d.nact, nsteps, conj, d.merged());
  } else {
    // runs without merged boundaries have a kernel of their own where the
    // other one's walk costs registers
    constexpr bool PLAIN = !merge_potential(SC::N, S, std::is_same<T, double>::value);
    auto k = PLAIN && d.mid < 0 ? k1d_prop_kernel<T, SC, S, 1, !PLAIN>
                                : k1d_prop_kernel<T, SC, S, 1>;
    const hipError_t e = set_lds((const void*)k, one);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3(count), dim3(SC::TPC), one, d.stream, (cx<T>*)psi,
                       (const cx<T>*)d.vexp, (const cx<T>*)d.kin, (const cx<T>*)d.tw[0],
                       d.prog_1d(), d.nact, nsteps, conj, d.merged());
  }
  return hipGetLastError();
}

template <typename T, class SC, int S>
hipError_t launch_obs(const DevView& d, const void* psi, const double* vraw, double ck,
                      double* out) {
  constexpr size_t one = (size_t)lds_pencil<SC>() * sizeof(cx<T>);
  auto k = k1d_obs_kernel<T, SC, S>;
  const hipError_t e = set_lds((const void*)k, one);
  if (e != hipSuccess) return e;
  TimedLaunch tl(d, KIND_OTHER,
                 S * SC::N * (sizeof(cx<T>) + (S + 1) / 2.0 * sizeof(double)));
  hipLaunchKernelGGL(k, dim3(1), dim3(SC::TPC), one, d.stream, (const cx<T>*)psi, vraw,
                     (const cx<T>*)d.tw[0], ck, out);
  return hipGetLastError();
}

template <class F>
hipError_t dispatch(int n, int S, bool f64, F&& f) {
#define SOP_1D_CASE(NN)                                                        \
  case NN:                                                                     \
    if (f64) {                                                                 \
      if (S == 1) return f.template operator()<double, S##NN, 1>();            \
      if (S == 2) return f.template operator()<double, S##NN, 2>();            \
    } else {                                                                   \
      if (S == 1) return f.template operator()<float, S##NN, 1>();             \
      if (S == 2) return f.template operator()<float, S##NN, 2>();             \
    }                                                                          \
    return hipErrorInvalidValue;
  switch (n) {
    SOP_1D_CASE(16)
    SOP_1D_CASE(32)
    SOP_1D_CASE(64)
    SOP_1D_CASE(128)
    SOP_1D_CASE(256)
    SOP_1D_CASE(512)
    SOP_1D_CASE(1024)
    SOP_1D_CASE(2048)
    SOP_1D_CASE(4096)
    SOP_1D_CASE(8192)
    default:
      return hipErrorInvalidValue;
  }
#undef SOP_1D_CASE
}

}  // namespace

bool k1d_supported(int n, int S) {
  if (S < 1 || S > 2) return false;
  switch (n) {
    case 16: case 32: case 64: case 128: case 256: case 512:
    case 1024: case 2048: case 4096: case 8192:
      return true;
    default:
      return false;
  }
}

hipError_t k1d_propagate(const DevView& d, void* psi, int64_t nsteps, int conj, int count) {
  if (d.timer) d.timer->break_chain();  // untimed work may precede this call
  return dispatch(d.n[0], d.S, d.f64, [&]<typename T, class SC, int S>() {
    return launch_prop<T, SC, S>(d, psi, nsteps, conj, count);
  });
}

hipError_t k1d_observe(const DevView& d, const void* psi, const double* vraw, double ck,
                       double* out) {
  if (d.timer) d.timer->break_chain();  // untimed work may precede this call
  return dispatch(d.n[0], d.S, d.f64, [&]<typename T, class SC, int S>() {
    return launch_obs<T, SC, S>(d, psi, vraw, ck, out);
  });
}

}  // namespace sop
