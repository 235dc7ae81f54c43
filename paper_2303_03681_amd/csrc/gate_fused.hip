// One two-qubit gate per workgroup, with the bond dimensions read from and
// written to device memory, so consecutive gates of a circuit queue on the
// stream without the host learning each new rank.  For bonds whose two-site
// matrix C~ is at most 128 x 128 (bond capacity <= 64 on both sides).
//
//   Eq. (C)   C = sum_{i'j'} Q B_q^{i'} B_{q+1}^{j'}          -> scratch (L2-resident)
//   Eq. (C~)  rows of lambda C, held in registers
//   LQ        larger ones: two LQ factorisations first (lq.hip says why)
//   Alg. 1    one-sided Jacobi on those rows until a sweep makes no rotation
//   Eq. (svd) sigma = row norms, stable descending order, truncation rank k
//   Eq. (Bl)  B_{q+1} <- V_k^+,  B_q <- C V_k / ||sigma_1..k||,  lambda <- sigma_k / ||sigma_1..k||
//
// Jacobi layout: 8 waves; wave w holds two blocks of 8 rows ("top" and
// "bottom"), each lane E elements of every row (e = lane + 64 k).  A sweep is
// a round-robin over the nb blocks: in round r the blocks at positions
// w and nb-1-w meet in wave w (position 0 fixed, the others advance by one),
// so every block pair meets once per sweep; round 0 also pairs the rows
// inside each block.  Within a wave the 64 cross pairs of its two blocks run
// as 8 sub-rounds of 8 disjoint pairs whose reductions interleave.  Between
// rounds, blocks move through LDS in two phases (tops, then bottoms), so at
// most nb/2 block slots are needed.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <utility>

#include "gemm_core.h"
#include "internal.h"
#include "jacobi_ops.h"
#include "lq_ops.h"
#include "wave_ops.h"

namespace mps {

namespace {

constexpr int FW = 8;      // waves per workgroup
constexpr int FB = 8;      // rows per block
constexpr int FMAXN = 128; // rows (2 D_l) and row length (2 D_r) limit
// Matrices of more elements (or more than twice as many rows as columns) are
// LQ-factorised before Algorithm 1.  A gate in us, factorised / directly, on random
// matrices graded over six decades: 16 x 16 116 / 94, 16 x 32 117 / 84, 24 x 24 214 /
// 192, 32 x 32 246 / 198, 64 x 64 503 / 455, but tall 32 x 16 150 / 204, 66 x 32 325 /
// 1,004, 60 x 14 149 / 664.  On the matrices of a UCCSD chain, whose rows are closer to
// parallel, it gains: 40 gates on 12 qubits D = 64 8.3 / 23.1 ms.  With the line at 512
// elements that step of the program takes 9.2 instead of 8.8 ms and one on ten-qubit
// fragments (32 x 32) 8.0 instead of 7.6.
constexpr int FPRE = 32 * 32;

// ---------------------------------------------------------------------------
// Eight pairs at a time.  The 16 per-lane partial sums (Re and Im of x^+y of 8
// pairs) are reduce-scattered over the wave (each lane ends with one full sum
// instead of all 16), so that lane l computes Algorithm 1's rotation of pair
// l & 7 (8 pairs per instruction stream); the coefficients then go to scalar
// registers for the vector updates.  The squared norms of the wave's 16 rows
// live in two registers, row l & 7 of the top and of the bottom block on lane
// l, fresh at every round and moved by +-t |b_ij| per rotation.
//
// What bounds it: instruction issue on one compute unit.  The pairings of a
// round are therefore loops over a few unrolled sub-rounds (rows move between
// registers instead), which keeps the kernel inside the 64 KB instruction
// cache that two compute units share: with all 15 sub-rounds of both register
// widths unrolled the code took 169 KB and a 128 x 128 sweep 650 us.

// Lane l receives lane (l + S) & 7 of a value that repeats every 8 lanes.
template <int S>
__device__ __forceinline__ double ror8(double x) {
  if constexpr (S % 8 == 0) return x;
  else return dpp_mov<0x120 + 8 - S % 8>(x);
}

// Row pairs of one group: pair i joins row xr(i) and row yr(i) of the 16 rows
// (0..7 top, 8..15 bottom).
template <int S>
struct CrossPairs {  // (top[i], bottom[(i + S) % 8])
  static constexpr int xr(int i) { return i; }
  static constexpr int yr(int i) { return FB + (i + S) % FB; }
};
struct IntraPairs {  // (position i, position 7 - i) inside the top (i < 4) and the bottom block
  static constexpr int xr(int i) { return i < 4 ? i : FB + i - 4; }
  static constexpr int yr(int i) { return i < 4 ? 7 - i : FB + 11 - i; }
};

template <int E, int R>
__device__ __forceinline__ double2 (&row(double2 (&T)[FB][E], double2 (&B)[FB][E]))[E] {
  if constexpr (R < FB) return T[R];
  else return B[R - FB];
}

template <int E, class P, int I>
__device__ __forceinline__ void partials_one(double2 (&T)[FB][E], double2 (&B)[FB][E], double (&v)[16]) {
  pair_partials_xy<E>(row<E, P::xr(I)>(T, B), row<E, P::yr(I)>(T, B), v[I], v[8 + I]);
}

template <int E, class P, int I>
__device__ __forceinline__ void apply_one(double2 (&T)[FB][E], double2 (&B)[FB][E], const Rot& mine) {
  Rot rt;  // row x plays a_i: x' = c x + s conj(e) y, y' = c y - s e x
  rt.c = readlane_d(mine.c, I);
  rt.ar = readlane_d(mine.ar, I);
  rt.ai = readlane_d(mine.ai, I);
  rt.br = -rt.ar;
  rt.bi = rt.ai;
  pair_apply<E>(row<E, P::xr(I)>(T, B), row<E, P::yr(I)>(T, B), rt);
}
template <int E, class P, int I>
__device__ __forceinline__ void apply_if(double2 (&T)[FB][E], double2 (&B)[FB][E], uint32_t act, const Rot& mine) {
  if ((act >> I) & 1) apply_one<E, P, I>(T, B, mine);
}

// Eight disjoint pairs: bxx, byy are the squared norms of lane l's pair
// (l & 7); *d receives t |b_ij| of the pairs that rotate (0 for the others).
template <int E, class P, int... I>
__device__ __forceinline__ int rot8(double2 (&T)[FB][E], double2 (&B)[FB][E], double bxx, double byy, double* d,
                                    double eps, double floor, int lane, std::integer_sequence<int, I...>) {
  double v[16];  // v[8c + i]: component c (0 Re, 1 Im) of x_i^+ y_i
  (partials_one<E, P, I>(T, B, v), ...);
  const double x = reduce_scatter16(v, lane);
  const double other = dpp_mov<0x128>(x);  // row_ror:8, the lane with the other component
  const bool im_lane = (lane >> 3) & 1;
  const double br = im_lane ? other : x, bi = im_lane ? x : other;
  const bool need = pair_needs_rot(bxx, byy, br, bi, eps, floor);
  const uint32_t act = (uint32_t)__ballot(need) & 0xFFu;
  *d = 0.0;
  if (act == 0) return 0;  // no pair rotates: skip the rotation formula
  Rot mine;
  double dn;
  pair_rot_coeffs(bxx, byy, br, bi, mine, &dn);
  *d = need ? dn : 0.0;
  const int rot = __popc(act);
  if (E == 1 && rot > 4) {
    // most pairs rotate: one straight run of all eight, the others by the
    // identity, instead of a branch per pair (two registers per row leave the
    // scheduler no room to interleave them)
    mine.c = need ? mine.c : 1.0;
    mine.ar = need ? mine.ar : 0.0;
    mine.ai = need ? mine.ai : 0.0;
    (apply_one<E, P, I>(T, B, mine), ...);
  } else {
    (apply_if<E, P, I>(T, B, act, mine), ...);
  }
  return rot;
}

template <int E, int S>
__device__ __forceinline__ int cross_sub(double2 (&T)[FB][E], double2 (&B)[FB][E], double& nt, double& nbm,
                                         double eps, double floor, int lane) {
  double d;
  const int rot = rot8<E, CrossPairs<S>>(T, B, nt, ror8<S>(nbm), &d, eps, floor, lane,
                                         std::make_integer_sequence<int, 8>{});
  nt += d;
  nbm -= ror8<8 - S>(d);
  return rot;
}

// The 64 pairs of the top and the bottom block: sub-rounds of eight disjoint
// pairs, four unrolled, then the halves of the bottom block change places
// (twice, so they end where they were).
template <int E>
__device__ __forceinline__ int cross_all(double2 (&T)[FB][E], double2 (&B)[FB][E], double& nt, double& nbm,
                                         double eps, double floor, int lane) {
  int rot = 0;
#pragma clang loop unroll(disable)
  for (int h = 0; h < 2; ++h) {
    rot += cross_sub<E, 0>(T, B, nt, nbm, eps, floor, lane);
    rot += cross_sub<E, 1>(T, B, nt, nbm, eps, floor, lane);
    rot += cross_sub<E, 2>(T, B, nt, nbm, eps, floor, lane);
    rot += cross_sub<E, 3>(T, B, nt, nbm, eps, floor, lane);
#pragma unroll
    for (int t = 0; t < FB / 2; ++t)
#pragma unroll
      for (int k = 0; k < E; ++k) {
        const double2 x = B[t][k];
        B[t][k] = B[t + FB / 2][k];
        B[t + FB / 2][k] = x;
      }
    nbm = ror8<4>(nbm);
  }
  return rot;
}

// The 28 pairs inside each block by the circle method: seven sub-rounds of
// (position i, position 7 - i), after each of which positions 1..7 advance by
// one (seven advances restore the order).
template <int E>
__device__ __forceinline__ int intra_all(double2 (&T)[FB][E], double2 (&B)[FB][E], double& nt, double& nbm,
                                         double eps, double floor, int lane) {
  int rot = 0;
  const int l8 = lane & 7;
  const bool low = l8 < 4;
  const int from = (lane & ~7) | (l8 == 0 ? 0 : (l8 == 7 ? 1 : l8 + 1));
#pragma clang loop unroll(disable)
  for (int s = 0; s < FB - 1; ++s) {
    // lane l < 4: pair (top l, top 7 - l); l >= 4: (bottom l - 4, bottom 11 - l)
    const double bs = ror8<4>(nbm);
    const double bxx = low ? nt : bs, byy = dpp_mov<0x141>(low ? bs : nt);  // half mirror: lane 7 - l
    double d;
    rot += rot8<E, IntraPairs>(T, B, bxx, byy, &d, eps, floor, lane, std::make_integer_sequence<int, 8>{});
    const double dm = dpp_mov<0x141>(d);
    nt += low ? d : -dm;
    nbm = ror8<4>(bs + (low ? -dm : d));
    nt = __shfl(nt, from, 64);
    nbm = __shfl(nbm, from, 64);
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const double2 t1 = T[1][k], b1 = B[1][k];
#pragma unroll
      for (int t = 1; t < FB - 1; ++t) {
        T[t][k] = T[t + 1][k];
        B[t][k] = B[t + 1][k];
      }
      T[FB - 1][k] = t1;
      B[FB - 1][k] = b1;
    }
  }
  return rot;
}

// Fresh squared norms of the 16 rows a wave holds.
template <int E>
__device__ __forceinline__ void row_norms(const double2 (&T)[FB][E], const double2 (&B)[FB][E], double& nt,
                                          double& nbm, int lane) {
  double v[2 * FB];
#pragma unroll
  for (int t = 0; t < FB; ++t) {
    double a = 0.0, b = 0.0;
#pragma unroll
    for (int k = 0; k < E; ++k) {
      a = norm_acc(T[t][k], a);
      b = norm_acc(B[t][k], b);
    }
    v[t] = a;
    v[FB + t] = b;
  }
  const double x = reduce_scatter16(v, lane), other = dpp_mov<0x128>(x);
  const bool bottom = (lane >> 3) & 1;
  nt = bottom ? other : x;
  nbm = bottom ? x : other;
}

template <int E>
__device__ __forceinline__ void blk_store(const double2 (&X)[FB][E], double2* slot, int lane) {
#pragma unroll
  for (int t = 0; t < FB; ++t)
#pragma unroll
    for (int k = 0; k < E; ++k) slot[(t * E + k) * 64 + lane] = X[t][k];
}

template <int E>
__device__ __forceinline__ void blk_load(double2 (&X)[FB][E], const double2* slot, int lane) {
#pragma unroll
  for (int t = 0; t < FB; ++t)
#pragma unroll
    for (int k = 0; k < E; ++k) X[t][k] = slot[(t * E + k) * 64 + lane];
}

// Advance the round-robin by one round: position p <- position p + 1 for
// p = 1 .. nb-2, position nb-1 <- position 1.  In waves: top(w) <- top(w+1)
// for 1 <= w <= nwa-2, top(nwa-1) <- bottom(nwa-1), bottom(w) <- bottom(w-1)
// for w >= 1, bottom(0) <- top(1); top(0) stays.  Every wave of the
// workgroup calls this (it holds the barriers).
template <int E>
__device__ __forceinline__ void advance(double2 (&T)[FB][E], double2 (&B)[FB][E], double2* xs,
                                        int wv, int nwa, int lane) {
  constexpr int SLOT = FB * 64 * E;
  __syncthreads();
  if (wv >= 1 && wv < nwa) blk_store<E>(T, xs + (size_t)(wv - 1) * SLOT, lane);
  __syncthreads();
  if (wv >= 1 && wv <= nwa - 2) blk_load<E>(T, xs + (size_t)wv * SLOT, lane);
  if (wv == nwa - 1) {
#pragma unroll
    for (int t = 0; t < FB; ++t)
#pragma unroll
      for (int k = 0; k < E; ++k) T[t][k] = B[t][k];
  }
  __syncthreads();
  if (wv <= nwa - 2) blk_store<E>(B, xs + (size_t)(wv + 1) * SLOT, lane);
  __syncthreads();
  if (wv >= 1 && wv < nwa) blk_load<E>(B, xs + (size_t)wv * SLOT, lane);
  if (wv == 0) blk_load<E>(B, xs, lane);
}

// Algorithm 1 on the rows held in T and B (nb blocks, positions as set up by
// the caller: wave w holds blocks w and nb-1-w): sweeps until one makes no
// rotation.  Returns the sweeps used, or 0 if max_sweeps were not enough.
// The block arrangement is the initial one again on return.  s_rot: two ints
// of shared memory, zero on entry.  Every thread of the workgroup calls this.
template <int E>
__device__ __forceinline__ int jacobi_sweeps(double2 (&T)[FB][E], double2 (&B)[FB][E], double2* xs,
                                             int* s_rot, int nb, int max_sweeps, double eps, double floor) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nwa = nb / 2;
  for (int sw = 0; sw < max_sweeps; ++sw) {
    int rot = 0;
    for (int r = 0; r < nb - 1; ++r) {
      if (wv < nwa) {
        // squared norms, fresh for every round and then tracked through its rotations
        double nt, nbm;
        row_norms<E>(T, B, nt, nbm, lane);
        if (r == 0) rot += intra_all<E>(T, B, nt, nbm, eps, floor, lane);
        rot += cross_all<E>(T, B, nt, nbm, eps, floor, lane);
      }
      if (nb > 2) advance<E>(T, B, xs, wv, nwa, lane);
    }
    if (lane == 0 && rot) atomicAdd(&s_rot[sw & 1], rot);
    __syncthreads();
    const int total = s_rot[sw & 1];
    __syncthreads();
    if (threadIdx.x == 0) s_rot[sw & 1] = 0;  // reused two sweeps on, after more barriers
    if (total == 0) return sw + 1;
  }
  return 0;
}

__device__ __forceinline__ void set_status(const FusedGate& g, int code) {
  g.status[1] = g.gate;
  __threadfence();
  g.status[0] = code;
}

}  // namespace

// Workgroup-shared scalars of one gate.
struct FusedShared {
  double sig[FMAXN];
  int perm[FMAXN];
  int rank[FMAXN];
  double part[FW];
  int rot[2];
  int k;
  double inv, least;
  int ok;
};

// Eq. (C): C[(i,a)][(j,r)] = sum_{i'j'} Q[2i+j][2i'+j'] (B_q^{i'} B_{q+1}^{j'})[a][r]
// A wave takes 16 a x 16 r of all four (i', j'), so that the gate mixes its
// accumulators.
__device__ __forceinline__ void gate_theta(const FusedGate& g, int Dl, int Dm, int Dr) {
  const int m = 2 * Dr;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const int ta = (Dl + 15) / 16, tr = (Dr + 15) / 16;
  for (int t = wv; t < ta * tr; t += FW) {
    const int a0 = (t / tr) * 16, r0 = (t % tr) * 16;
    const double2* pa = g.bq + (size_t)min(a0 + lr, Dl - 1) * Dm;
    const double2* pb = g.bq1 + min(r0 + lr, Dr - 1);
    d4_t re[2][2], im[2][2];
    wave_gemm<double, 2, 2>(
        re, im, Dm, [&](int i, int k) { return pa[(size_t)i * Dl * Dm + k]; },
        [&](int j, int k) { return pb[(size_t)j * Dm * Dr + (size_t)k * Dr]; });
    const int r = r0 + lr;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int a = a0 + acc_row<double>(lk, v);
      if (a >= Dl || r >= Dr) continue;
#pragma unroll
      for (int ij = 0; ij < 4; ++ij) {
        double2 acc = make_double2(0.0, 0.0);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const double2 u = g.u[ij * 4 + k];
          const double tx = re[k >> 1][k & 1][v], ty = im[k >> 1][k & 1][v];
          acc.x += u.x * tx - u.y * ty;
          acc.y += u.x * ty + u.y * tx;
        }
        g.c[(size_t)((ij >> 1) * Dl + a) * m + (ij & 1) * Dr + r] = acc;
      }
    }
  }
  __syncthreads();
}

// One LQ factorisation by the whole workgroup (rows x len, RPW rows per
// wave): load(i, e) is element e of row i; the orthonormal rows go to q_out
// (len each; may be null) and the adjoint factor to f_out (rows x rows).  All
// rows are in registers before anything is written, so f_out may be where
// they came from.
template <int E, int RPW, class Load>
__device__ __forceinline__ void gate_lq(int rows, int len, double2* xs, double2* q_out, double2* f_out, Load load) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double2 x[RPW][E];
#pragma unroll
  for (int a = 0; a < RPW; ++a) {
    const int i = a * FW + wv;
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int e = lane + 64 * k;
      x[a][k] = i < rows && e < len ? load(i, e) : make_double2(0.0, 0.0);
    }
  }
  __syncthreads();
  mgs_rows<E, FW, RPW>(
      x, rows, xs, 0.0, [&](int t, double r) { f_out[(size_t)t * rows + t] = make_double2(r, 0.0); },
      [&](int t, const double2* q) {
        if (q_out)
          for (int e = threadIdx.x; e < len; e += FW * 64) q_out[(size_t)t * len + e] = q[e];
        for (int i = threadIdx.x; i < t; i += FW * 64) f_out[(size_t)t * rows + i] = make_double2(0.0, 0.0);
      },
      [&](int t, int u, double re, double im) { f_out[(size_t)t * rows + u] = make_double2(re, -im); });
  __syncthreads();
}

// Register layout by size: 64 elements of a row per lane register, 64 rows per
// 8 rows of a wave.
template <class Load>
__device__ __forceinline__ void gate_lq_any(int rows, int len, double2* xs, double2* q_out, double2* f_out,
                                            Load load) {
  if (rows <= 64 && len <= 64) gate_lq<1, 8>(rows, len, xs, q_out, f_out, load);
  else if (rows <= 64) gate_lq<2, 8>(rows, len, xs, q_out, f_out, load);
  else gate_lq<2, 16>(rows, len, xs, q_out, f_out, load);
}

// Algorithm 1 on n rows of length m (load(row, e)), then sigma_i = ||row_i||,
// stable descending order and truncation (sh.sig, perm, rank, k, inv; sh.ok).
// store(row, rank, e, value / sigma) is called for the kept rows.  False, with
// the status set, if it did not converge or is not finite.
template <int E, class Load, class Store>
__device__ __forceinline__ bool gate_svd(const FusedGate& g, double2* xs, FusedShared& sh, int n, int m, int capk,
                                         Load load, Store store) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int nb = (n + FB - 1) / FB;
  nb = nb < 2 ? 2 : nb + (nb & 1);
  const int nwa = nb / 2;
  double2 T[FB][E], B[FB][E];
  double part = 0.0;
  {
    const int gt = wv * FB, gb = (nb - 1 - wv) * FB;
#pragma unroll
    for (int t = 0; t < FB; ++t)
#pragma unroll
      for (int k = 0; k < E; ++k) {
        const int e = lane + 64 * k;
        double2 vt = make_double2(0.0, 0.0), vb = make_double2(0.0, 0.0);
        if (wv < nwa && e < m) {
          if (gt + t < n) vt = load(gt + t, e);
          if (gb + t < n) vb = load(gb + t, e);
        }
        T[t][k] = vt;
        B[t][k] = vb;
        part += vt.x * vt.x + vt.y * vt.y + vb.x * vb.x + vb.y * vb.y;
      }
  }
  part = wave_sum(part);
  if (lane == 0) sh.part[wv] = part;
  if (threadIdx.x == 0) {
    sh.rot[0] = 0;
    sh.rot[1] = 0;
  }
  __syncthreads();
  double fro2 = 0.0;
#pragma unroll
  for (int w = 0; w < FW; ++w) fro2 += sh.part[w];
  if (!isfinite(fro2)) {
    if (threadIdx.x == 0) set_status(g, 1);
    return false;
  }
  const double eps = g.eps_scale * (double)m;
  const double floor = eps * eps * fro2;
  const int done = jacobi_sweeps<E>(T, B, xs, sh.rot, nb, g.max_sweeps, eps, floor);
  if (!done) {
    if (threadIdx.x == 0) set_status(g, 2);
    return false;
  }

  {
    double nt, nbm;
    row_norms<E>(T, B, nt, nbm, lane);
    if (wv < nwa && lane < 2 * FB) {
      const int row = lane < FB ? wv * FB + lane : (nb - 1 - wv) * FB + (lane - FB);
      if (row < n) sh.sig[row] = sqrt(lane < FB ? nt : nbm);
    }
  }
  if (threadIdx.x < FMAXN) sh.perm[threadIdx.x] = threadIdx.x;
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += FW * 64) {
    const double si = sh.sig[i];
    int rk = 0;
    for (int j = 0; j < n; ++j) {
      const double sj = sh.sig[j];
      rk += (sj > si) || (sj == si && j < i);
    }
    sh.perm[rk] = i;
    sh.rank[i] = rk;
  }
  __syncthreads();
  if (wv == 0) {  // lane l: the l-th and the (l + 64)-th largest
    const double s0 = lane < n ? sh.sig[sh.perm[lane]] : 0.0;
    const double s1 = lane + 64 < n ? sh.sig[sh.perm[lane + 64]] : 0.0;
    const double tot = wave_sum(s0 * s0 + s1 * s1), cut = g.cutoff * sqrt(tot);
    int k = __popcll(__ballot(lane < n && s0 > cut)) + __popcll(__ballot(lane + 64 < n && s1 > cut));
    k = min(max(k, 1), capk);
    const double kept2 = wave_sum((lane < k ? s0 * s0 : 0.0) + (lane + 64 < k ? s1 * s1 : 0.0));
    const double disc2 = wave_sum((lane < k ? 0.0 : s0 * s0) + (lane + 64 < k ? 0.0 : s1 * s1));
    const double kept = sqrt(kept2);
    if (lane == 0) {
      sh.ok = isfinite(tot) && kept > 0.0 && isfinite(kept);
      sh.inv = sh.ok ? 1.0 / kept : 0.0;
      sh.k = k;
      sh.least = 0x1p-53 * sqrt(tot);  // no vector for round-off (finalize_kernel says why)
      if (sh.ok) {
        *g.disc += tot > 0.0 ? disc2 / tot : 0.0;
        *g.sweeps += done;
      } else {
        set_status(g, 1);
      }
    }
  }
  __syncthreads();
  if (!sh.ok) return false;
  if (wv < nwa) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int base = h == 0 ? wv * FB : (nb - 1 - wv) * FB;
#pragma unroll
      for (int t = 0; t < FB; ++t) {
        const int row = base + t;
        if (row >= n) continue;
        const int p = sh.rank[row];
        if (p >= sh.k) continue;
        const double sv = sh.sig[row];
        const double is = sv > sh.least ? 1.0 / sv : 0.0;
#pragma unroll
        for (int kk = 0; kk < E; ++kk) {
          const int e = lane + 64 * kk;
          if (e < m) {
            const double2 x = h == 0 ? T[t][kk] : B[t][kk];
            store(p, e, make_double2(x.x * is, x.y * is));
          }
        }
      }
    }
  }
  return true;
}

// V^+ (k x m) = Z Q, Z (k x na) and Q (na x m) in memory, as the right site
// tensor [j][p][r].
__device__ __forceinline__ void gate_vec(const FusedGate& g, const double2* z, const double2* q, int k, int na, int m,
                                         int Dr) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const int tp = (k + 15) / 16, te = (m + 15) / 16;
  for (int t = wv; t < tp * te; t += FW) {
    const int p0 = (t / te) * 16, e0 = (t % te) * 16;
    const double2* pa = z + (size_t)min(p0 + lr, k - 1) * na;
    const double2* pb = q + min(e0 + lr, m - 1);
    d4_t re[1][1], im[1][1];
    wave_gemm<double, 1, 1>(
        re, im, na, [&](int, int s) { return pa[s]; }, [&](int, int s) { return pb[(size_t)s * m]; });
    const int e = e0 + lr, j = e >= Dr ? 1 : 0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int p = p0 + acc_row<double>(lk, v);
      if (p < k && e < m)
        g.bq1[((size_t)j * k + p) * Dr + e - j * Dr] = make_double2(re[0][0][v], im[0][0][v]);
    }
  }
  __syncthreads();
}

// The rows of that V^+ (orthonormal to eps sigma_1 / sigma_p) orthonormalised
// in order, in place.
template <int E, int RPW>
__device__ __forceinline__ void gate_orth(const FusedGate& g, double2* xs, int k, int m, int Dr) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double2 x[RPW][E];
#pragma unroll
  for (int a = 0; a < RPW; ++a)
#pragma unroll
    for (int c = 0; c < E; ++c) {
      const int e = lane + 64 * c, p = a * FW + wv, j = e >= Dr ? 1 : 0;
      x[a][c] = p < k && e < m ? g.bq1[((size_t)j * k + p) * Dr + e - j * Dr] : make_double2(0.0, 0.0);
    }
  __syncthreads();
  mgs_rows<E, FW, RPW>(
      x, k, xs, kDependent, [](int, double) {},
      [&](int t, const double2* v) {
        for (int e = threadIdx.x; e < m; e += FW * 64) {
          const int j = e >= Dr ? 1 : 0;
          g.bq1[((size_t)j * k + t) * Dr + e - j * Dr] = v[e];
        }
      },
      [](int, int, double, double) {});
  __syncthreads();
}

// Eq. (Bl): B_q[(i,a)][p] = inv sum_e C[(i,a)][e] conj(V^+[p][e]), V^+ from the
// right site tensor [j][p][r]; 2 x 2 tiles per wave where there are enough.
template <int MT, int NT>
__device__ __forceinline__ void gate_left(const FusedGate& g, int n, int k, int m, int Dr, double inv) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const int tm = (n + 16 * MT - 1) / (16 * MT), tn = (k + 16 * NT - 1) / (16 * NT);
  for (int t = wv; t < tm * tn; t += FW) {
    const int i0 = (t / tn) * 16 * MT, p0 = (t % tn) * 16 * NT;
    const double2* pa[MT];
    const double2* pb[NT];
#pragma unroll
    for (int i = 0; i < MT; ++i) pa[i] = g.c + (size_t)min(i0 + 16 * i + lr, n - 1) * m;
#pragma unroll
    for (int j = 0; j < NT; ++j) pb[j] = g.bq1 + (size_t)min(p0 + 16 * j + lr, k - 1) * Dr;
    const size_t half = (size_t)k * Dr - Dr;  // from element e of block 0 to element e of block 1
    d4_t re[MT][NT], im[MT][NT];
    wave_gemm<double, MT, NT>(
        re, im, m, [&](int i, int e) { return pa[i][e]; },
        [&](int j, int e) {
          const double2 v = pb[j][e >= Dr ? half + e : e];
          return make_double2(v.x, -v.y);
        });
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = i0 + 16 * i + acc_row<double>(lk, v), p = p0 + 16 * j + lr;
          if (row < n && p < k)
            g.bq[(size_t)row * k + p] = make_double2(re[i][j][v] * inv, im[i][j][v] * inv);
        }
  }
}

// One two-qubit gate by the whole workgroup; xs is the dynamic LDS (block
// slots, rows in flight).  Every thread returns at the same point.
__device__ __forceinline__ void gate_any(const FusedGate& g, double2* xs, FusedShared& sh) {
  if (g.status[0] != 0) return;  // an earlier gate of this run failed: apply nothing
  const int Dl = g.dims[g.q], Dm = g.dims[g.q + 1], Dr = g.dims[g.q + 2];
  const int n = 2 * Dl, m = 2 * Dr;
  const double2* C = g.c;
  gate_theta(g, Dl, Dm, Dr);
  const int capk = min(g.cap_k, min(n, m));

  // Eq. (C~) is lambda_a C[(i,a)]; i and a exchanged, its rows are in the order of lambda
  const bool pre = g.l1 != nullptr && (n * m > FPRE || n > 2 * m);
  if (pre) {
    // Two LQ factorisations before Algorithm 1, as for the batched gates: the
    // sweeps then see a nearly diagonal matrix (UCCSD chains: 14.6 -> 5.6
    // sweeps on average), and V^+ is their result times the first Q.
    double2* f = g.l1;   // factors, then Z
    double2* q1 = g.l2;  // Q of the first factorisation
    const int na = min(n, m);
    if (n > m) {  // tall: its m x m triangular factor has the same right vectors
      gate_lq_any(m, n, xs, nullptr, f, [&](int i, int e) {
        const double l = g.lam_l[e % Dl];
        const double2 v = C[(size_t)e * m + i];
        return make_double2(l * v.x, -l * v.y);
      });
      gate_lq_any(m, m, xs, q1, f, [&](int i, int e) { return f[(size_t)i * m + e]; });
    } else {
      gate_lq_any(n, m, xs, q1, f, [&](int i, int e) {
        const int a = i >> 1;
        const double l = g.lam_l[a];
        const double2 v = C[(size_t)((i & 1) * Dl + a) * m + e];
        return make_double2(l * v.x, l * v.y);
      });
    }
    gate_lq_any(na, na, xs, nullptr, f, [&](int i, int e) { return f[(size_t)i * na + e]; });
    auto load = [&](int i, int e) { return f[(size_t)i * na + e]; };
    auto store = [&](int p, int e, double2 v) { f[(size_t)p * na + e] = v; };
    if (!(na <= 64 ? gate_svd<1>(g, xs, sh, na, na, capk, load, store)
                   : gate_svd<2>(g, xs, sh, na, na, capk, load, store)))
      return;
    __syncthreads();
    gate_vec(g, f, q1, sh.k, na, m, Dr);
    if (m <= 64) gate_orth<1, 8>(g, xs, sh.k, m, Dr);
    else if (sh.k <= 64) gate_orth<2, 8>(g, xs, sh.k, m, Dr);
    else gate_orth<2, 16>(g, xs, sh.k, m, Dr);
  } else {
    auto load = [&](int i, int e) {
      const double l = g.lam_l[i % Dl];
      const double2 v = C[(size_t)i * m + e];
      return make_double2(l * v.x, l * v.y);
    };
    auto store = [&](int p, int e, double2 v) {
      const int j = e >= Dr ? 1 : 0;
      g.bq1[((size_t)j * sh.k + p) * Dr + e - j * Dr] = v;
    };
    if (!(m <= 64 ? gate_svd<1>(g, xs, sh, n, m, capk, load, store)
                  : gate_svd<2>(g, xs, sh, n, m, capk, load, store)))
      return;
  }
  const int k = sh.k;
  const double inv = sh.inv;

  // ---- Eq. (Bl): lambda_{q+1} <- sigma_k / ||sigma_k||
  for (int p = threadIdx.x; p < k; p += FW * 64) g.lam_m[p] = sh.sig[sh.perm[p]] * inv;

  __syncthreads();
  if (n > 64 || k > 32) gate_left<2, 2>(g, n, k, m, Dr, inv);
  else gate_left<1, 1>(g, n, k, m, Dr, inv);
  if (threadIdx.x == 0) g.dims[g.q + 1] = k;
}

__global__ __launch_bounds__(FW * 64) void gate2q_fused_kernel(FusedGate g) {
  extern __shared__ double2 xs[];
  __shared__ FusedShared sh;
  gate_any(g, xs, sh);
}

// One step of several gate lists: workgroup f applies gate g0 + step of run
// f (Eq. 1q in place, or a two-qubit gate by gate_any) unless its list is
// exhausted or an earlier gate of the run failed.  The host enqueues the
// steps in order on one stream.
__global__ __launch_bounds__(FW * 64) void fused_step_kernel(const FusedRun* runs, int64_t step) {
  extern __shared__ double2 xs[];
  __shared__ FusedShared sh;
  const FusedRun r = runs[blockIdx.x];
  const int64_t gi = r.g0 + step;
  if (gi >= r.g1 || r.status[0] != 0) return;
  const int q = r.q0[gi];
  const double2* u = r.u + (size_t)gi * 16;
  if (r.q1[gi] < 0) {
    double2* b = r.sites[q];
    const int count = r.dims[q] * r.dims[q + 1];
    const double2 u00 = u[0], u01 = u[1], u10 = u[2], u11 = u[3];
    for (int i = threadIdx.x; i < count; i += FW * 64) {
      const double2 x0 = b[i], x1 = b[count + i];
      const double2 a = cmul(u00, x0), bb = cmul(u01, x1), c = cmul(u10, x0), d = cmul(u11, x1);
      b[i] = make_double2(a.x + bb.x, a.y + bb.y);
      b[count + i] = make_double2(c.x + d.x, c.y + d.y);
    }
    return;
  }
  const FusedGate g{r.sites[q], r.sites[q + 1], r.lam[q], r.lam[q + 1], u, r.dims, r.c, r.l1, r.l2, r.status,
                    r.disc, r.sweeps, q, (int)gi, r.cap[q + 1], r.max_sweeps, r.cutoff, r.eps_scale};
  gate_any(g, xs, sh);
}

// Eq. (1q) with the bond dimensions read on the device.
__global__ void gate1q_dev_kernel(double2* b, const double2* u, const int* dims, const int* status,
                                  int q) {
  if (status[0] != 0) return;
  const int count = dims[q] * dims[q + 1];
  const double2 u00 = u[0], u01 = u[1], u10 = u[2], u11 = u[3];
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += gridDim.x * blockDim.x) {
    const double2 x0 = b[i], x1 = b[count + i];
    const double2 a = cmul(u00, x0), bb = cmul(u01, x1), c = cmul(u10, x0), d = cmul(u11, x1);
    b[i] = make_double2(a.x + bb.x, a.y + bb.y);
    b[count + i] = make_double2(c.x + d.x, c.y + d.y);
  }
}

// Algorithm 1 alone on matrices of at most 128 rows of at most 128 complex
// elements (one workgroup per item, all sweeps in one launch): rows it.w
// (n x m, row-major) are rotated in place; *it.sweeps_done receives the
// sweeps used, or -max_sweeps if they were not enough; ||w||_F^2 is read
// from *it.fro2.
template <int E>
__device__ __forceinline__ void jacobi_small_body(const JacItem& it, int max_sweeps, double eps_scale,
                                                  double2* xs, int* s_rot) {
  const int n = it.n, m = it.m;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int nb = (n + FB - 1) / FB;
  nb = nb < 2 ? 2 : nb + (nb & 1);
  const int nwa = nb / 2;
  double2 T[FB][E], B[FB][E];
#pragma unroll
  for (int t = 0; t < FB; ++t)
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int e = lane + 64 * k, rt = wv * FB + t, rb = (nb - 1 - wv) * FB + t;
      const bool ok = wv < nwa && e < m;
      T[t][k] = ok && rt < n ? it.w[(size_t)rt * m + e] : make_double2(0.0, 0.0);
      B[t][k] = ok && rb < n ? it.w[(size_t)rb * m + e] : make_double2(0.0, 0.0);
    }
  const double eps = eps_scale * (double)m;
  const double floor = eps * eps * (*it.fro2);
  const int done = jacobi_sweeps<E>(T, B, xs, s_rot, nb, max_sweeps, eps, floor);
  if (wv < nwa) {
#pragma unroll
    for (int t = 0; t < FB; ++t)
#pragma unroll
      for (int k = 0; k < E; ++k) {
        const int e = lane + 64 * k, rt = wv * FB + t, rb = (nb - 1 - wv) * FB + t;
        if (e < m) {
          if (rt < n) it.w[(size_t)rt * m + e] = T[t][k];
          if (rb < n) it.w[(size_t)rb * m + e] = B[t][k];
        }
      }
  }
  if (threadIdx.x == 0) *it.sweeps_done = done > 0 ? done : -max_sweeps;
}

__global__ __launch_bounds__(FW * 64) void jacobi_small_kernel(const JacItem* items, int max_sweeps,
                                                               double eps_scale) {
  extern __shared__ double2 xs[];
  __shared__ int s_rot[2];
  const JacItem it = items[blockIdx.x];
  if (threadIdx.x == 0) {
    s_rot[0] = 0;
    s_rot[1] = 0;
  }
  __syncthreads();
  if (it.m <= 64) jacobi_small_body<1>(it, max_sweeps, eps_scale, xs, s_rot);
  else jacobi_small_body<2>(it, max_sweeps, eps_scale, xs, s_rot);
}

size_t fused_lds_bytes() { return (size_t)FW * FB * 64 * 2 * sizeof(double2); }

hipError_t configure_fused_lds() {
  hipError_t e = hipFuncSetAttribute((const void*)gate2q_fused_kernel,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)fused_lds_bytes());
  if (e != hipSuccess) return e;
  e = hipFuncSetAttribute((const void*)fused_step_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)fused_lds_bytes());
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute((const void*)jacobi_small_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)fused_lds_bytes());
}

hipError_t launch_gate2q_fused(const FusedGate& g, int max_len, hipStream_t s) {
  if (max_len > FMAXN) return hipErrorInvalidValue;
  hipLaunchKernelGGL(gate2q_fused_kernel, dim3(1), dim3(FW * 64), fused_lds_bytes(), s, g);
  return hipGetLastError();
}

hipError_t launch_fused_step(const FusedRun* runs_dev, int n_runs, int64_t step, hipStream_t s) {
  if (n_runs <= 0) return hipSuccess;
  hipLaunchKernelGGL(fused_step_kernel, dim3(n_runs), dim3(FW * 64), fused_lds_bytes(), s, runs_dev,
                     step);
  return hipGetLastError();
}

hipError_t launch_jacobi_small(const JacItem* items_dev, int items, int max_sweeps, double eps_scale,
                               hipStream_t s) {
  if (items <= 0) return hipSuccess;
  hipLaunchKernelGGL(jacobi_small_kernel, dim3(items), dim3(FW * 64), fused_lds_bytes(), s, items_dev,
                     max_sweeps, eps_scale);
  return hipGetLastError();
}

hipError_t launch_gate1q_dev(double2* b, const double2* u, const int* dims, const int* status, int q,
                             int max_count, hipStream_t s) {
  const int blocks = std::max(1, std::min(64, (max_count + 255) / 256));
  hipLaunchKernelGGL(gate1q_dev_kernel, dim3(blocks), dim3(256), 0, s, b, u, dims, status, q);
  return hipGetLastError();
}

}  // namespace mps
