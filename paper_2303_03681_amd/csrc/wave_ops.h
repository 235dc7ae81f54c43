// Wave-level helpers shared by the device kernels (64-lane wavefronts).
#pragma once

#include <hip/hip_runtime.h>

namespace mps {

// Row pointers of the work matrices are global memory: typed so, the loads
// and stores are global (not flat) instructions with immediate offsets.
typedef double __attribute__((ext_vector_type(2))) dvec2;
typedef __attribute__((address_space(1))) dvec2 gdvec2;

// Lane permutation within rows of 16 lanes (DPP control CTRL) of a double.
// Every control used stays inside the row, so no lane keeps an old value and
// none has to be set up.
template <int CTRL>
__device__ __forceinline__ double dpp_mov(double x) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}

// v + (v of lane ^ 16) and v + (v of lane ^ 32), by the row and half-wave
// swaps of gfx950 (vector instructions; the LDS crossbar path of a shuffle
// takes several times their latency).  Both partners add in the same order.
__device__ __forceinline__ double add_xor16(double v) {
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
__device__ __forceinline__ double add_xor32(double v) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}

// Barrier of the workgroup that orders LDS accesses only: __syncthreads() also
// waits until every earlier store to memory has landed (hundreds of cycles in
// a loop that stores a result per step).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// 1 / sqrt(x) for positive normal x: the hardware estimate and two Newton steps.
__device__ __forceinline__ double rsqrt_newton(double x) {
  double y = __builtin_amdgcn_rsq(x);
  double h = 0.5 * x * y;
  y = fma(y, fma(-h, y, 0.5), y);
  h = 0.5 * x * y;
  return fma(y, fma(-h, y, 0.5), y);
}

__device__ __forceinline__ double readlane_d(double x, int l) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(x), l);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(x), l);
  return __hiloint2double(hi, lo);
}

// A wave-uniform value moved to scalar registers (it is identical in all lanes).
__device__ __forceinline__ double wave_uniform(double x) {
  const int lo = __builtin_amdgcn_readfirstlane(__double2loint(x));
  const int hi = __builtin_amdgcn_readfirstlane(__double2hiint(x));
  return __hiloint2double(hi, lo);
}

// Sum over the 64 lanes of a wave, the same bits in every lane (each step
// adds a and b in both orders, and a + b == b + a exactly): DPP moves within
// rows of 16 lanes, then two cross-row swaps.
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_mov<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_mov<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_mov<0x141>(v);  // row_half_mirror
  v += dpp_mov<0x140>(v);  // row_mirror
  return add_xor32(add_xor16(v));
}

// wave_sum of N independent values, stage by stage so the N dependency
// chains interleave (the same bits as N separate wave_sum calls).
template <int N>
__device__ __forceinline__ void wave_sum_n(double (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_mov<0xB1>(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_mov<0x4E>(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_mov<0x141>(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_mov<0x140>(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = add_xor16(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = add_xor32(v[i]);
}

// acc + conj(a) b in two chains of fused multiply-adds.
__device__ __forceinline__ void dot_acc(double2 a, double2 b, double& re, double& im) {
  re = fma(a.y, b.y, fma(a.x, b.x, re));
  im = fma(-a.y, b.x, fma(a.x, b.y, im));
}

// x - (cr + i ci) q
__device__ __forceinline__ void sub_mul(double2& x, double cr, double ci, double2 q) {
  x.x = fma(ci, q.y, fma(-cr, q.x, x.x));
  x.y = fma(-ci, q.x, fma(-cr, q.y, x.y));
}

__device__ __forceinline__ double norm_acc(double2 a, double s) { return fma(a.y, a.y, fma(a.x, a.x, s)); }

// Sums of N = 2, 4 or 8 values over the wave, handed back in scalar registers:
// reduce-scattered over lane bit 3 (2 for N >= 4, 1 for N = 8), so that every lane
// carries one sum through the remaining steps, then read from the lane that
// holds it.  About half the instructions of wave_sum_n for these N.
template <int N>
__device__ __forceinline__ void wave_sum_scalar(double (&v)[N], int lane) {
  static_assert(N == 2 || N == 4 || N == 8, "N sums");
  double a[N / 2], x;
  const bool h3 = (lane >> 3) & 1, h2 = (lane >> 2) & 1, h1 = (lane >> 1) & 1;
#pragma unroll
  for (int j = 0; j < N / 2; ++j)
    a[j] = (h3 ? v[N / 2 + j] : v[j]) + dpp_mov<0x140>(h3 ? v[j] : v[N / 2 + j]);  // row_mirror
  if constexpr (N == 2) {
    x = a[0] + dpp_mov<0x141>(a[0]);
    x += dpp_mov<0x4E>(x);
  } else {
    double b[N / 4];
#pragma unroll
    for (int j = 0; j < N / 4; ++j)
      b[j] = (h2 ? a[N / 4 + j] : a[j]) + dpp_mov<0x141>(h2 ? a[j] : a[N / 4 + j]);  // row_half_mirror
    if constexpr (N == 8) x = (h1 ? b[1] : b[0]) + dpp_mov<0x4E>(h1 ? b[0] : b[1]);  // quad_perm [2,3,0,1]
    else x = b[0] + dpp_mov<0x4E>(b[0]);
  }
  x += dpp_mov<0xB1>(x);  // quad_perm [1,0,3,2]
  x = add_xor32(add_xor16(x));
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int l = i * (16 / N);  // lane bits 3.. hold the index of the sum
    v[i] = readlane_d(x, l);
  }
}

// One reduce-scatter stage: keep the half of v selected by this lane's bit,
// add the partner's copy of it (the partner keeps the other half).
template <int H>
__device__ __forceinline__ double rs_pick(const double (&v)[2 * H], int j, bool hi, bool send) {
  return (hi != send) ? v[H + j] : v[j];
}

// The full sum of v[l & 15] on lane l: lane bits 3, 2, 1, 0 by DPP, then full
// sums over bits 4 and 5 (the same bits in every lane that holds a sum).
__device__ __forceinline__ double reduce_scatter16(const double (&v)[16], int lane) {
  double v8[8], v4[4], v2[2];
  const bool h3 = (lane >> 3) & 1, h2 = (lane >> 2) & 1, h1 = (lane >> 1) & 1, h0 = lane & 1;
#pragma unroll
  for (int j = 0; j < 8; ++j) v8[j] = rs_pick<8>(v, j, h3, false) + dpp_mov<0x140>(rs_pick<8>(v, j, h3, true));
#pragma unroll
  for (int j = 0; j < 4; ++j) v4[j] = rs_pick<4>(v8, j, h2, false) + dpp_mov<0x141>(rs_pick<4>(v8, j, h2, true));
#pragma unroll
  for (int j = 0; j < 2; ++j) v2[j] = rs_pick<2>(v4, j, h1, false) + dpp_mov<0x4E>(rs_pick<2>(v4, j, h1, true));
  const double x = rs_pick<1>(v2, 0, h0, false) + dpp_mov<0xB1>(rs_pick<1>(v2, 0, h0, true));
  return add_xor32(add_xor16(x));
}

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

}  // namespace mps
