// kernels_aux.hip -- evolution-operator table formation and FP64 reductions.
//
// Potential tables (Sec. "Pruning splitting coefficients": the unique
// evolution operators are computed once at initialisation; Sec. "Molecular
// Hamiltonian in the diabatic basis": the exponential of the S x S potential
// matrix from its Jacobi diagonalisation).  Per grid point the real
// symmetric V(q) is diagonalised by cyclic two-sided Jacobi rotations in
// FP64; for every unique coefficient c the complex-symmetric
// exp(-i tau V/hbar) = R diag(exp(-i lambda tau/hbar)) R^T, tau = c dt, is
// formed in FP64 and rounded once to the plan precision; its packed upper
// triangle is stored structure-of-arrays, [unique][entry][point] for 1D
// grids, or tile-contiguous for the 3D z-pass ([unique][tile][z][entry][col]).
//
// Reductions: surface populations of an FP64 state, <psi|phi> and distances
// (the observables' sums with <T> are in kernels_1d.hip and kernels_3d.hip,
// with the transforms they need); every sum is FP64 with a fixed block
// count and a fixed-order tree, so results are bitwise reproducible.
#include <algorithm>

#include "eigen.hpp"
#include "fft_core.hpp"
#include "internal.hpp"

namespace sop {
namespace {

// Destination index of (table u, entry e, point x): structure of arrays for
// 1D (tile = 0, or -W with the points in wave order) or the z-pass tile layout
// for a cubic 3D grid of side n (x below 2^31: 32-bit divisions).
__device__ __forceinline__ int64_t table_index(int64_t npts, int NE, int tile, int n, int u, int e,
                                               int64_t x) {
  if (tile <= 0)
    return ((int64_t)u * NE + e) * npts + (tile == 0 ? x : (int64_t)wave_order_x(-tile, (int)x));
  const uint32_t row = (uint32_t)x / (uint32_t)n, xx = (uint32_t)x - row * (uint32_t)n;
  const uint32_t z = row / (uint32_t)n, y = row - z * (uint32_t)n;
  const uint32_t tx = xx / (uint32_t)tile;
  const uint32_t tl = y * ((uint32_t)n / (uint32_t)tile) + tx;
  return (int64_t)u * NE * npts + (int64_t)tl * ((int64_t)n * NE * tile) +
         ((int64_t)z * NE + e) * tile + (xx - tx * (uint32_t)tile);
}

template <typename T, int S>
__global__ void __launch_bounds__(256)
    k_form_vexp(const double* __restrict__ vraw, int64_t npts, const double* __restrict__ taus,
                int ntau, int tile, int n, cx<T>* __restrict__ out,
                const double* __restrict__ dtab, unsigned dmask,
                const double* __restrict__ s_dev) {
  constexpr int NE = S * (S + 1) / 2;
  const double sd = dmask ? *s_dev : 0.0;  // driven: V = vraw + s D
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < npts;
       x += (int64_t)gridDim.x * blockDim.x) {
    double A[S][S], R[S][S];
    int e = 0;
#pragma unroll
    for (int i = 0; i < S; ++i)
#pragma unroll
      for (int j = i; j < S; ++j) {
        const int64_t o = (int64_t)e * npts + x;
        const double vij = (dmask >> e) & 1 ? vraw[o] + sd * dtab[o] : vraw[o];
        A[i][j] = vij;
        A[j][i] = vij;
        ++e;
      }
    jacobi_sym<S>(A, R);
    for (int u = 0; u < ntau; ++u) {
      double ere[S], eim[S];
#pragma unroll
      for (int l = 0; l < S; ++l) sincos(-A[l][l] * taus[u], &eim[l], &ere[l]);
      int ee = 0;
#pragma unroll
      for (int i = 0; i < S; ++i)
#pragma unroll
        for (int j = i; j < S; ++j) {
          double re = 0.0, im = 0.0;
#pragma unroll
          for (int l = 0; l < S; ++l) {
            const double rr = R[i][l] * R[j][l];
            re += rr * ere[l];
            im += rr * eim[l];
          }
          const int64_t o = table_index(npts, NE, tile, n, u, ee, x);
          if constexpr (sizeof(T) == 8) {
            out[o] = cx<T>{(T)re, (T)im};
          } else {  // FP32: the pair (rounded, residue) at index 2 o
            const float hr = (float)re, hi = (float)im;
            out[2 * o] = cx<float>{hr, hi};
            out[2 * o + 1] = cx<float>{(float)(re - (double)hr), (float)(im - (double)hi)};
          }
          ++ee;
        }
    }
  }
}

// Block-level fixed-order sum of NV values per thread; thread 0 writes the
// block's NV sums to out.
template <int NV>
__device__ void block_sum(double (&acc)[NV], double* out) {
  __shared__ double red[kReduceThreads][NV];
  const int tid = threadIdx.x;
#pragma unroll
  for (int v = 0; v < NV; ++v) red[tid][v] = acc[v];
  __syncthreads();
  for (int w = kReduceThreads / 2; w > 0; w >>= 1) {
    if (tid < w) {
#pragma unroll
      for (int v = 0; v < NV; ++v) red[tid][v] += red[tid + w][v];
    }
    __syncthreads();
  }
  if (tid == 0) {
#pragma unroll
    for (int v = 0; v < NV; ++v) out[v] = red[0][v];
  }
}

// Per block: sum_x |psi_s(x)|^2 for each s.
template <int S>
__global__ void __launch_bounds__(kReduceThreads)
    k_populations(const cx<double>* __restrict__ psi, int64_t npts,
                  double* __restrict__ partials) {
  double acc[S];
#pragma unroll
  for (int s = 0; s < S; ++s) acc[s] = 0.0;
  for (int64_t x = (int64_t)blockIdx.x * kReduceThreads + threadIdx.x; x < npts;
       x += (int64_t)gridDim.x * kReduceThreads) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const cx<double> p = psi[s * npts + x];
      acc[s] += p.re * p.re + p.im * p.im;
    }
  }
  block_sum<S>(acc, partials + (size_t)blockIdx.x * S);
}

template <typename T>
__global__ void __launch_bounds__(kReduceThreads)
    k_overlap(const cx<T>* __restrict__ a, const cx<T>* __restrict__ b, int64_t n,
              double* __restrict__ partials) {
  double acc[2] = {0.0, 0.0};
  for (int64_t i = (int64_t)blockIdx.x * kReduceThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kReduceThreads) {
    const cx<T> p = a[i], q = b[i];
    // conj(p) q
    acc[0] += (double)p.re * (double)q.re + (double)p.im * (double)q.im;
    acc[1] += (double)p.re * (double)q.im - (double)p.im * (double)q.re;
  }
  block_sum<2>(acc, partials + (size_t)blockIdx.x * 2);
}

// sum |a - b|^2 and sum |b|^2, the difference taken in FP64 from the
// stored values.
template <typename T>
__global__ void __launch_bounds__(kReduceThreads)
    k_distance(const cx<T>* __restrict__ a, const cx<T>* __restrict__ b, int64_t n,
               double* __restrict__ partials) {
  double acc[2] = {0.0, 0.0};
  for (int64_t i = (int64_t)blockIdx.x * kReduceThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kReduceThreads) {
    const cx<T> p = a[i], q = b[i];
    const double dr = (double)p.re - (double)q.re, di = (double)p.im - (double)q.im;
    acc[0] += dr * dr + di * di;
    acc[1] += (double)q.re * (double)q.re + (double)q.im * (double)q.im;
  }
  block_sum<2>(acc, partials + (size_t)blockIdx.x * 2);
}

// Sums nblocks rows of nv partials in a fixed order into out[nv].
__global__ void __launch_bounds__(kReduceThreads)
    k_final(const double* __restrict__ partials, int nblocks, int nv, double* __restrict__ out) {
  __shared__ double red[kReduceThreads];
  for (int v = 0; v < nv; ++v) {
    double acc = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += kReduceThreads) acc += partials[(size_t)b * nv + v];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = kReduceThreads / 2; w > 0; w >>= 1) {
      if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
      __syncthreads();
    }
    if (threadIdx.x == 0) out[v] = red[0];
    __syncthreads();
  }
}

// Compact eigen form of V(q) for the FP64 3D z-pass (S = 2, 3): per point
// the rotation R of V = R diag(lam) R^T (det R = +1, a product of Jacobi
// rotations) and the eigenvalues, in eig_slots(S) complex slots of the
// z-pass tile layout: S = 3 as the unit quaternion (w, x) (y, z) of R and
// (lam_0, lam_1) (lam_2, 0); S = 2 as (cos, sin) of the rotation angle and
// (lam_0, lam_1).  One table serves every coefficient: each potential
// action forms exp(-i tau lam) itself.  The quaternion is the row of products
// with its largest component (largest of w^2, x^2, y^2, z^2, each =
// (1 +- R_00 +- R_11 +- R_22)/4), scaled to unit length.
template <int S>
__global__ void __launch_bounds__(256)
    k_form_eigq(const double* __restrict__ vraw, int64_t npts, int tile, int n,
                cx<double>* __restrict__ out, const double* __restrict__ dtab, unsigned dmask,
                const double* __restrict__ s_dev) {
  constexpr int NQ = eig_slots(S);
  const double sd = dmask ? *s_dev : 0.0;  // driven: V = vraw + s D
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < npts;
       x += (int64_t)gridDim.x * blockDim.x) {
    double A[S][S], R[S][S];
    int e = 0;
#pragma unroll
    for (int i = 0; i < S; ++i)
#pragma unroll
      for (int j = i; j < S; ++j) {
        const int64_t o = (int64_t)e * npts + x;
        const double vij = (dmask >> e) & 1 ? vraw[o] + sd * dtab[o] : vraw[o];
        A[i][j] = vij;
        A[j][i] = vij;
        ++e;
      }
    jacobi_sym<S>(A, R);
    cx<double> slot[NQ];
    eig_form_slots<S>(A, R, slot);
#pragma unroll
    for (int q = 0; q < NQ; ++q) out[table_index(npts, NQ, tile, n, 0, q, x)] = slot[q];
  }
}

// Eigen-decomposition table for the adjoint of one surface: per point the pair
// (R = 1, V) in the z-pass tile layout (two and three surfaces use the compact
// eigen form of k_form_eigq).  Written for any S: R row-major S x S, then the
// eigenvalues, as S(S+1)/2 pairs of doubles.
template <int S>
__global__ void __launch_bounds__(256)
    k_form_eig(const double* __restrict__ vraw, int64_t npts, int tile, int n,
               cx<double>* __restrict__ out) {
  constexpr int NE = S * (S + 1) / 2;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < npts;
       x += (int64_t)gridDim.x * blockDim.x) {
    double A[S][S], R[S][S];
    int e = 0;
#pragma unroll
    for (int i = 0; i < S; ++i)
#pragma unroll
      for (int j = i; j < S; ++j) {
        const double vij = vraw[(int64_t)e * npts + x];
        A[i][j] = vij;
        A[j][i] = vij;
        ++e;
      }
    jacobi_sym<S>(A, R);
    double flat[2 * NE];
#pragma unroll
    for (int i = 0; i < S; ++i)
#pragma unroll
      for (int j = 0; j < S; ++j) flat[i * S + j] = R[i][j];
#pragma unroll
    for (int l = 0; l < S; ++l) flat[S * S + l] = A[l][l];
#pragma unroll
    for (int q = 0; q < NE; ++q)
      out[table_index(npts, NE, tile, n, 0, q, x)] = cx<double>{flat[2 * q], flat[2 * q + 1]};
  }
}

// vraw = vbase + sum_k delta_k dv_k (the potential is linear in its parameters);
// grid (blocks, packed entries).  Bound by its bytes: 128^3 x 3 with three
// couplings, all entries of dv read 80 us, the nonzero ones 42 us.
__global__ void __launch_bounds__(256)
    k_vparams(double* __restrict__ vraw, const double* __restrict__ vbase,
              const double* __restrict__ dv, EntryMasks mask, const double* __restrict__ delta,
              int nparams, int64_t npts) {
  const int64_t e0 = (int64_t)blockIdx.y * npts;
  const int64_t table = (int64_t)gridDim.y * npts;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < npts;
       x += (int64_t)gridDim.x * blockDim.x) {
    double v = vbase[e0 + x];
    for (int k = 0; k < nparams; ++k)
      if ((mask.m[k] >> blockIdx.y) & 1) v += delta[k] * dv[k * table + e0 + x];
    vraw[e0 + x] = v;
  }
}

// lambda_s = w_s psi_s (seed of the adjoint sweep for L = sum_s w_s P_s).
__global__ void __launch_bounds__(256)
    k_scale_surfaces(cx<double>* __restrict__ lam, const cx<double>* __restrict__ psi,
                     const double* __restrict__ w, int S, int64_t npts) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < (int64_t)S * npts;
       i += (int64_t)gridDim.x * blockDim.x) {
    const double ws = w[i / npts];
    lam[i] = cx<double>{ws * psi[i].re, ws * psi[i].im};
  }
}

__global__ void __launch_bounds__(256) k_zero(double* __restrict__ p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0.0;
}

// Per block: g_k = sum_x sum_e Q_e(x) dv[k][e][x], k < NP, with Q_e(x) read
// from the accumulator's tile layout [tile (y, x/C)][z][e][x % C] on an n^3
// grid (point x = (z n + y) n + x0).  Bound by its bytes, of which the zero
// entries of dv were most (128^3 x 3, three couplings: 102 -> 40 us).
template <int NP>
__global__ void __launch_bounds__(kReduceThreads)
    k_grad_partials(const double* __restrict__ qacc, const double* __restrict__ dv,
                    EntryMasks mask, int NE, int64_t npts, int n, int cols, double* __restrict__ partials) {
  double acc[NP];
#pragma unroll
  for (int k = 0; k < NP; ++k) acc[k] = 0.0;
  const int64_t plane = (int64_t)n * n;
  for (int64_t x = (int64_t)blockIdx.x * kReduceThreads + threadIdx.x; x < npts;
       x += (int64_t)gridDim.x * kReduceThreads) {
    const int64_t z = x / plane, r = x - z * plane;
    const int64_t y = r / n, x0 = r - y * n;
    const int64_t qb = ((y * (n / cols) + x0 / cols) * n + z) * (int64_t)NE * cols + x0 % cols;
    for (int e = 0; e < NE; ++e) {
      const double q = qacc[qb + (int64_t)e * cols];
#pragma unroll
      for (int k = 0; k < NP; ++k)
        if ((mask.m[k] >> e) & 1) acc[k] += q * dv[((int64_t)k * NE + e) * npts + x];
    }
  }
  block_sum<NP>(acc, partials + (size_t)blockIdx.x * NP);
}

template <int S, typename T>
hipError_t form_impl(const DevView& d, const double* vraw, const double* taus, int ntau, int tile,
                     void* out, const double* dtab, unsigned dmask, const double* s_dev) {
  int blocks = (int)((d.npts + 255) / 256);
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL((k_form_vexp<T, S>), dim3(blocks), dim3(256), 0, d.stream, vraw, d.npts,
                     taus, ntau, tile, d.n[0], (cx<T>*)out, dtab, dmask, s_dev);
  return hipGetLastError();
}

}  // namespace

hipError_t form_vexp(const DevView& d, const double* vraw_dev, const double* taus, int ntau,
                     int tile, void* out, const double* dtab, unsigned dmask, const double* s_dev) {
  switch (d.S) {
    case 1: return d.f64 ? form_impl<1, double>(d, vraw_dev, taus, ntau, tile, out, dtab, dmask, s_dev)
                         : form_impl<1, float>(d, vraw_dev, taus, ntau, tile, out, dtab, dmask, s_dev);
    case 2: return d.f64 ? form_impl<2, double>(d, vraw_dev, taus, ntau, tile, out, dtab, dmask, s_dev)
                         : form_impl<2, float>(d, vraw_dev, taus, ntau, tile, out, dtab, dmask, s_dev);
    case 3: return d.f64 ? form_impl<3, double>(d, vraw_dev, taus, ntau, tile, out, dtab, dmask, s_dev)
                         : form_impl<3, float>(d, vraw_dev, taus, ntau, tile, out, dtab, dmask, s_dev);
    default: return hipErrorInvalidValue;
  }
}

hipError_t form_eigq(const DevView& d, const double* vraw_dev, int tile, void* out,
                     const double* dtab, unsigned dmask, const double* s_dev) {
  int blocks = (int)((d.npts + 255) / 256);
  if (blocks > 4096) blocks = 4096;
  cx<double>* o = (cx<double>*)out;
  switch (d.S) {
    case 2: hipLaunchKernelGGL(k_form_eigq<2>, dim3(blocks), dim3(256), 0, d.stream, vraw_dev, d.npts, tile, d.n[0], o, dtab, dmask, s_dev); break;
    case 3: hipLaunchKernelGGL(k_form_eigq<3>, dim3(blocks), dim3(256), 0, d.stream, vraw_dev, d.npts, tile, d.n[0], o, dtab, dmask, s_dev); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t form_eig(const DevView& d, const double* vraw_dev, int tile, void* out) {
  int blocks = (int)((d.npts + 255) / 256);
  if (blocks > 4096) blocks = 4096;
  switch (d.S) {
    case 1: hipLaunchKernelGGL(k_form_eig<1>, dim3(blocks), dim3(256), 0, d.stream, vraw_dev, d.npts, tile, d.n[0], (cx<double>*)out); break;
    // two and three surfaces: the compact eigen form (rotation and eigenvalues)
    case 2:
    case 3: return form_eigq(d, vraw_dev, tile, out);
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t set_vparams(const DevView& d, double* vraw, const double* vbase, const double* dv,
                       const EntryMasks& mask, const double* delta_dev, int nparams) {
  const int blocks = (int)std::min<int64_t>(1024, (d.npts + 255) / 256);
  hipLaunchKernelGGL(k_vparams, dim3(blocks, d.S * (d.S + 1) / 2), dim3(256), 0, d.stream, vraw,
                     vbase, dv, mask, delta_dev, nparams, d.npts);
  return hipGetLastError();
}

hipError_t adjoint_seed(const DevView& d, void* lam, const void* psi, const double* w_dev,
                        double* qacc) {
  hipLaunchKernelGGL(k_scale_surfaces, dim3(2048), dim3(256), 0, d.stream, (cx<double>*)lam,
                     (const cx<double>*)psi, w_dev, d.S, d.npts);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_zero, dim3(2048), dim3(256), 0, d.stream, qacc,
                     (int64_t)d.S * (d.S + 1) / 2 * d.npts);
  return hipGetLastError();
}

hipError_t grad_reduce(const DevView& d, const double* qacc, int cols, const double* dv,
                       const EntryMasks& nonzero, int nparams, double* partials,
                       double* out_dev) {
  if (d.ndim != 3 || cols <= 0 || d.n[0] % cols != 0) return hipErrorInvalidValue;
  const int NE = d.S * (d.S + 1) / 2;
  // a table of zeros keeps one entry, so that a sum over invalid (NaN) values
  // is NaN for it too
  EntryMasks mask = nonzero;
  for (unsigned& m : mask.m) m |= m == 0;
  switch (nparams) {
#define SOP_GRAD_CASE(K)                                                                    \
  case K:                                                                                   \
    hipLaunchKernelGGL(k_grad_partials<K>, dim3(kReduceBlocks), dim3(kReduceThreads), 0,    \
                       d.stream, qacc, dv, mask, NE, d.npts, d.n[0], cols, partials);       \
    break;
    SOP_GRAD_CASE(1)
    SOP_GRAD_CASE(2)
    SOP_GRAD_CASE(3)
    SOP_GRAD_CASE(4)
    SOP_GRAD_CASE(5)
    SOP_GRAD_CASE(6)
    SOP_GRAD_CASE(7)
    SOP_GRAD_CASE(8)
#undef SOP_GRAD_CASE
    default:
      return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_final, dim3(1), dim3(kReduceThreads), 0, d.stream, partials, kReduceBlocks,
                     nparams, out_dev);
  return hipGetLastError();
}

hipError_t pops_reduce(const DevView& d, const void* psi, double* partials, double* out_dev) {
  auto k = d.S == 1 ? k_populations<1> : d.S == 2 ? k_populations<2> : k_populations<3>;
  if (!d.f64 || d.S < 1 || d.S > 3) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k, dim3(kReduceBlocks), dim3(kReduceThreads), 0, d.stream,
                     (const cx<double>*)psi, d.npts, partials);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_final, dim3(1), dim3(kReduceThreads), 0, d.stream, partials, kReduceBlocks,
                     d.S, out_dev);
  return hipGetLastError();
}

hipError_t distance_reduce(const DevView& d, const void* psi, const void* phi, double* partials,
                           double* out_dev) {
  const int64_t n = d.npts * d.S;
  if (d.f64)
    hipLaunchKernelGGL(k_distance<double>, dim3(kReduceBlocks), dim3(kReduceThreads), 0,
                       d.stream, (const cx<double>*)psi, (const cx<double>*)phi, n, partials);
  else
    hipLaunchKernelGGL(k_distance<float>, dim3(kReduceBlocks), dim3(kReduceThreads), 0,
                       d.stream, (const cx<float>*)psi, (const cx<float>*)phi, n, partials);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_final, dim3(1), dim3(kReduceThreads), 0, d.stream, partials, kReduceBlocks,
                     2, out_dev);
  return hipGetLastError();
}

hipError_t overlap_reduce(const DevView& d, const void* psi, const void* phi, double* partials,
                          double* out_dev) {
  const int64_t n = d.npts * d.S;
  if (d.f64)
    hipLaunchKernelGGL(k_overlap<double>, dim3(kReduceBlocks), dim3(kReduceThreads), 0, d.stream,
                       (const cx<double>*)psi, (const cx<double>*)phi, n, partials);
  else
    hipLaunchKernelGGL(k_overlap<float>, dim3(kReduceBlocks), dim3(kReduceThreads), 0, d.stream,
                       (const cx<float>*)psi, (const cx<float>*)phi, n, partials);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_final, dim3(1), dim3(kReduceThreads), 0, d.stream, partials, kReduceBlocks,
                     2, out_dev);
  return hipGetLastError();
}

}  // namespace sop
