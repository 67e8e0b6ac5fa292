// reduce.hpp -- fixed-order FP64 sums of a workgroup.
#pragma once

#include <hip/hip_runtime.h>

namespace sop {

// Sums of NV values over the NT threads of a workgroup (NT a power of two up
// to 64, or a multiple of 64): lane exchanges inside each wave, then the
// waves' sums in order through `red` (NV * NT / 64 doubles).  Every thread of
// the first wave receives the sums.  The order is fixed, so results are
// bitwise reproducible.  `red` may hold anything that all threads have read;
// the barrier before its writes keeps those reads ahead.
template <int NT, int NV>
__device__ __forceinline__ void workgroup_sum(double (&a)[NV], double* red) {
  constexpr int W = NT < 64 ? NT : 64;
#pragma unroll
  for (int off = W / 2; off > 0; off >>= 1)
#pragma unroll
    for (int k = 0; k < NV; ++k) a[k] += __shfl_xor(a[k], off);
  if constexpr (NT > 64) {
    const int w = (int)threadIdx.x / 64;
    __syncthreads();
    if (threadIdx.x % 64 == 0) {
#pragma unroll
      for (int k = 0; k < NV; ++k) red[NV * w + k] = a[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      double s = 0.0;
      for (int i = 0; i < NT / 64; ++i) s += red[NV * i + k];
      a[k] = s;
    }
  }
}

}  // namespace sop
