// Modified Gram-Schmidt on rows held in the registers of one workgroup, shared
// by the blocked LQ kernels and the fused gate.
#pragma once

#include <hip/hip_runtime.h>

#include "wave_ops.h"

namespace mps {

// `least` of the pass that orthonormalises V^+.  Its rows have unit norm and
// overlap with the rows before by eps sigma_1 / sigma_p, so one of which less
// than 1e-4 is left has a sigma_p that is round-off (kept where the cutoff is
// below it).  Normalised, what is left is the rounding of the subtraction --
// parallel to an earlier row where the rows have one element, which would count
// that direction twice.
constexpr double kDependent = 1e-8;

// Row u of `rows` sits on wave u % NW in slot u / NW, lane + 64 k holding
// element k.  Row t is normalised at step t and taken out of the later rows.
// buf: 2 x 64 E elements of shared memory; diag(t, r) is called by one lane
// with the row's norm, done(t, q) by every thread with the finished row in
// shared memory, coef(t, u, re, im) by one lane with q_t^+ x_u (u > t).
// The owner hands its row on through one of two buffers, so that there is one
// barrier per step: a buffer is rewritten two steps later, after every wave
// has passed the barrier in between.  The barriers order LDS only: what done
// and coef store in memory is visible to the workgroup after its next
// __syncthreads().  Every thread of the workgroup calls this.
// What bounds it is instruction issue, not the chain: at 64 rows of 64
// elements a step takes 0.97 us, about what the reductions of eight rows per
// wave issue; handing the next row on ahead of the others (look-ahead) took
// 1.26 us.
template <int E, int NW, int RPW, class Diag, class Done, class Coef>
__device__ __forceinline__ void mgs_rows(double2 (&x)[RPW][E], int rows, double2* buf, double least, Diag diag,
                                         Done done, Coef coef) {
  constexpr int G = RPW < 4 ? RPW : 4;  // rows whose products are reduced together
  static_assert(RPW % G == 0, "whole groups");
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int t = 0; t < rows; ++t) {
    double2* b = buf + (size_t)(t & 1) * 64 * E;
    if (wv == t % NW) {
#pragma unroll
      for (int a = 0; a < RPW; ++a) {
        if (a != t / NW) continue;
        double nn = 0.0;
#pragma unroll
        for (int k = 0; k < E; ++k) nn = norm_acc(x[a][k], nn);
        nn = wave_sum(nn);
        const double inv = nn > least ? rsqrt_newton(nn) : (nn <= least ? 0.0 : nn);  // NaN stays NaN
#pragma unroll
        for (int k = 0; k < E; ++k) b[lane + 64 * k] = make_double2(x[a][k].x * inv, x[a][k].y * inv);
        if (lane == 0) diag(t, nn * inv);
      }
    }
    lds_barrier();
    done(t, b);
    if (wv + (RPW - 1) * NW <= t) continue;  // no later row on this wave
    double2 q[E];
#pragma unroll
    for (int k = 0; k < E; ++k) q[k] = b[lane + 64 * k];
#pragma unroll
    for (int g = 0; g < RPW; g += G) {
      if (wv + (g + G - 1) * NW <= t) continue;
      double c[2 * G];
#pragma unroll
      for (int a = 0; a < G; ++a) {
        c[2 * a] = c[2 * a + 1] = 0.0;
#pragma unroll
        for (int k = 0; k < E; ++k) dot_acc(q[k], x[g + a][k], c[2 * a], c[2 * a + 1]);
      }
      wave_sum_scalar<2 * G>(c, lane);
#pragma unroll
      for (int a = 0; a < G; ++a) {
        const int u = (g + a) * NW + wv;
        if (u <= t || u >= rows) continue;  // done, or padding
#pragma unroll
        for (int k = 0; k < E; ++k) sub_mul(x[g + a][k], c[2 * a], c[2 * a + 1], q[k]);
        if (lane == 0) coef(t, u, c[2 * a], c[2 * a + 1]);
      }
    }
  }
}

}  // namespace mps
