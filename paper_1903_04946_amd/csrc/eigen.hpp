// eigen.hpp -- eigen-decomposition of the S x S potential matrix of a point.
#pragma once

#include "fft_core.hpp"
#include "internal.hpp"

namespace sop {

// 1/sqrt(x) for a normal x: the hardware's estimate (about 24 bits) and one
// third-order step, e = 1 - x y^2, y (1 + e/2 + 3 e^2/8): what is left is that
// step's rounding.  (The general square root and division spend most of their
// instructions on scaling and special cases.)
__device__ __forceinline__ double rsqrt_short(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-(x * y), y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

// Cyclic Jacobi rotations on a real symmetric S x S matrix (the upper
// triangle of A is used).  On return A is diagonal (eigenvalues on the
// diagonal) and R holds the eigenvectors in its columns.  Each rotation has
// tan(2 theta) = 2 a_pq / (a_qq - a_pp), |theta| <= pi/4 (the symmetric Schur
// step of Golub and Van Loan, Matrix Computations, Sec. 8.5), from two inverse
// square roots: with d = a_qq - a_pp, b = 2 a_pq sign(d) and y = 1/sqrt(d^2 + b^2),
//   cos 2 theta = |d| y,  sin 2 theta = b y,  1/c = 1/sqrt((1 + cos 2 theta)/2),
//   s = sin 2 theta / (2 c),  tan theta = s / c,
// and a_pp - t a_pq, a_qq + t a_pq on the diagonal.  The matrix is first
// scaled by the power of two that brings its largest entry to [1/2, 1), so
// that d^2 + b^2 neither overflows nor, with entries below 1e-150 of the
// largest taken as zero, underflows.
// The formation is bound by FP64 issue, then by its bytes: k_form_eigq at
// 128^3 x 3 with three couplings took 147 us with general divisions and
// square roots (three and two a rotation) and two-sided updates of the full
// matrix, and takes 80 us (44 us with one coupling, 5.4 TB/s).
template <int S>
__device__ __forceinline__ void jacobi_sym(double (&A)[S][S], double (&R)[S][S]) {
#pragma unroll
  for (int i = 0; i < S; ++i)
#pragma unroll
    for (int j = 0; j < S; ++j) R[i][j] = (i == j) ? 1.0 : 0.0;
  if constexpr (S == 1) return;
  double big = 0.0;
#pragma unroll
  for (int i = 0; i < S; ++i)
#pragma unroll
    for (int j = i; j < S; ++j) big = fmax(big, fabs(A[i][j]));
  const int ex = __builtin_amdgcn_frexp_exp(big);
#pragma unroll
  for (int i = 0; i < S; ++i)
#pragma unroll
    for (int j = i; j < S; ++j) A[i][j] = __builtin_amdgcn_ldexp(A[i][j], -ex);
  for (int sweep = 0; sweep < 24; ++sweep) {
    bool rotated = false;
#pragma unroll
    for (int p = 0; p < S - 1; ++p) {
#pragma unroll
      for (int q = p + 1; q < S; ++q) {
        const double apq = A[p][q], app = A[p][p], aqq = A[q][q];
        // negligible next to the diagonal or to the whole matrix
        if (fabs(apq) <= fmax(1e-18 * (fabs(app) + fabs(aqq)), 1e-150)) {
          A[p][q] = 0.0;
          continue;
        }
        rotated = true;
        const double d = aqq - app;
        const double b = d < 0.0 ? -2.0 * apq : 2.0 * apq;
        double c, s, t;
        if constexpr (S == 2) {
          // one rotation a point, the kernel waits for memory: correctly
          // rounded roots and quotients, t = b / (|d| + sqrt(d^2 + b^2))
          t = b / (fabs(d) + sqrt(fma(d, d, b * b)));
          c = 1.0 / sqrt(fma(t, t, 1.0));
          s = t * c;
        } else {
          const double y = rsqrt_short(fma(d, d, b * b));
          const double c2 = fma(0.5 * fabs(d), y, 0.5);  // cos^2 theta, in [1/2, 1]
          const double ci = rsqrt_short(c2);
          c = c2 * ci;
          s = (0.5 * (b * y)) * ci;
          t = s * ci;
        }
        A[p][p] = fma(-t, apq, app);
        A[q][q] = fma(t, apq, aqq);
        A[p][q] = 0.0;
#pragma unroll
        for (int r = 0; r < S; ++r) {
          if (r != p && r != q) {
            double& arp = r < p ? A[r][p] : A[p][r];
            double& arq = r < q ? A[r][q] : A[q][r];
            const double vp = arp, vq = arq;
            arp = fma(c, vp, -(s * vq));
            arq = fma(s, vp, c * vq);
          }
          const double rp = R[r][p], rq = R[r][q];
          R[r][p] = fma(c, rp, -(s * rq));
          R[r][q] = fma(s, rp, c * rq);
        }
      }
    }
    if (!rotated) break;
  }
#pragma unroll
  for (int i = 0; i < S; ++i) A[i][i] = __builtin_amdgcn_ldexp(A[i][i], ex);
}

// The eigen_slots(S) slots of the compact eigen form (kernels_aux.hip) from
// what jacobi_sym leaves in A and R.
template <int S>
__device__ __forceinline__ void eig_form_slots(const double (&A)[S][S], const double (&R)[S][S],
                                               cx<double> (&slot)[eig_slots(S)]) {
  if constexpr (S == 2) {
    slot[0] = cx<double>{R[0][0], R[1][0]};
    slot[1] = cx<double>{A[0][0], A[1][1]};
  } else {
    const double t0 = 1.0 + R[0][0] + R[1][1] + R[2][2];  // 4 w^2
    const double t1 = 1.0 + R[0][0] - R[1][1] - R[2][2];  // 4 x^2
    const double t2 = 1.0 - R[0][0] + R[1][1] - R[2][2];  // 4 y^2
    const double t3 = 1.0 - R[0][0] - R[1][1] + R[2][2];  // 4 z^2
    // 4 times the products with the largest component, chosen without
    // branches: (w^2, wx, wy, wz), (wx, x^2, xy, xz), ..
    const double wx = R[2][1] - R[1][2], wy = R[0][2] - R[2][0], wz = R[1][0] - R[0][1];
    const double xy = R[0][1] + R[1][0], xz = R[0][2] + R[2][0], yz = R[1][2] + R[2][1];
    const bool b0 = t0 >= t1 && t0 >= t2 && t0 >= t3;
    const bool b1 = !b0 && t1 >= t2 && t1 >= t3;
    const bool b2 = !b0 && !b1 && t2 >= t3;
    double w = b0 ? t0 : b1 ? wx : b2 ? wy : wz;
    double qx = b0 ? wx : b1 ? t1 : b2 ? xy : xz;
    double qy = b0 ? wy : b1 ? xy : b2 ? t2 : yz;
    double qz = b0 ? wz : b1 ? xz : b2 ? yz : t3;
    // scaled to a unit quaternion (the largest product is at least 1)
    const double nrm = rsqrt_short(fma(w, w, fma(qx, qx, fma(qy, qy, qz * qz))));
    slot[0] = cx<double>{w * nrm, qx * nrm};
    slot[1] = cx<double>{qy * nrm, qz * nrm};
    slot[2] = cx<double>{A[0][0], A[1][1]};
    slot[3] = cx<double>{A[2][2], 0.0};
  }
}

}  // namespace sop
