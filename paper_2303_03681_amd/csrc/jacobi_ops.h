// Algorithm 1's pair step on register-resident rows, shared by the Jacobi
// kernels: partial sums of x^+y per lane, the rotation test and the rotation
// of one pair from the reduced sums, and its application.
#pragma once

#include <hip/hip_runtime.h>

#include "wave_ops.h"

namespace mps {

struct Rot {
  double c, ar, ai, br, bi;  // x' = c x + (ar + i ai) y,  y' = c y + (br + i bi) x
};

// Algorithm 1's rotation test: |b_ij| > floor and |b_ij| > eps sqrt(b_ii
// b_jj), compared in squares (symmetric in the two rows).
__device__ __forceinline__ bool pair_needs_rot(double bxx, double byy, double br, double bi, double eps,
                                               double floor) {
  const double mag2 = br * br + bi * bi;
  return mag2 > floor * floor && mag2 > eps * eps * (bxx * byy);
}

// Algorithm 1's rotation from b_ii = bxx, b_jj = byy and b_ij of a pair that
// passed the test, row x playing a_i.  With w = 1 / sqrt(1 + tau^2) the
// formulas for t, c and s reduce to
//   c^2 = (1 + |tau| w) / 2,   s = sign(tau) w / (2 c),   t = s / c,
// three reciprocal square roots (of |b_ij|^2, 1 + tau^2 and c^2) where t and
// c as written take two, a square root and a division.  |tau| is capped where
// the rotation no longer changes anything.  *dn receives t |b_ij|, by which
// b_ii grows and b_jj shrinks.
__device__ __forceinline__ void pair_rot_coeffs(double bxx, double byy, double br, double bi, Rot& rt, double* dn) {
  const double delta = bxx - byy;
  const double mag2 = br * br + bi * bi;
  const double rinv = rsqrt_newton(mag2);  // 1 / |b_ij|
  const double at = fmin(fabs(delta) * (0.5 * rinv), 1e100);
  const double w = rsqrt_newton(fma(at, at, 1.0));
  const double c2 = fma(0.5 * at, w, 0.5);
  const double rc = rsqrt_newton(c2);  // 1 / c
  const double s = delta >= 0.0 ? 0.5 * w * rc : -0.5 * w * rc;
  rt.c = c2 * rc;
  // e = b_ij / |b_ij|;  a_i' = c a_i + s conj(e) a_j,  a_j' = c a_j - s e a_i
  rt.ar = s * (br * rinv);
  rt.ai = -s * (bi * rinv);
  rt.br = -rt.ar;
  rt.bi = rt.ai;
  *dn = s * rc * (mag2 * rinv);
}

// Partial sums of Re and Im of x^+y over this lane's elements.
template <int E>
__device__ __forceinline__ void pair_partials_xy(const double2 (&x)[E], const double2 (&y)[E],
                                                 double& re, double& im) {
  re = 0.0;
  im = 0.0;
#pragma unroll
  for (int k = 0; k < E; ++k) dot_acc(x[k], y[k], re, im);
}

template <int E>
__device__ __forceinline__ void pair_apply(double2 (&x)[E], double2 (&y)[E], const Rot& rt) {
#pragma unroll
  for (int k = 0; k < E; ++k) {
    const double2 a = x[k], b = y[k];
    x[k] = make_double2(rt.c * a.x + (rt.ar * b.x - rt.ai * b.y), rt.c * a.y + (rt.ar * b.y + rt.ai * b.x));
    y[k] = make_double2(rt.c * b.x + (rt.br * a.x - rt.bi * a.y), rt.c * b.y + (rt.br * a.y + rt.bi * a.x));
  }
}

}  // namespace mps
