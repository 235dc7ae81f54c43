// Device kernels of the MPS energy evaluation (gfx950).
//
//   init_product     product state B^s = delta_{s,b} (Methods, UCC: HF reference)
//   gate1q           Eq. (1q)
//   theta + mix      Eq. (C) as one batched MFMA GEMM, then the 4x4 gate mix and
//                    the lambda row scale of Eq. (C~)
//   jacobi_*         Algorithm 1 (one-sided Jacobi), block-parallel round-robin
//   finalize         sigma_i = ||a_i||, stable descending sort, truncation,
//                    normalised vectors -> B~_{q+1} = V (Eq. Bl) or canonical tensors
//   trunc            Eq. (Bl): B~_q = C V^+, an MFMA GEMM
//   canon_*          the GEMMs of the two canonicalisation sweeps
//   env_gemm, env_small  Eq. (expec2) transfer update L' = sum sigma A^{s+} L A^{s'}
//   gram, gram_pairs closing traces Tr(L R): tiles of (prefix, suffix) pairs at a
//                    bond, or the needed pairs alone
//   energy           compensated FP64 sum_k c_k <P_k> in string order
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <mutex>
#include <type_traits>
#include <vector>

#include "gemm_core.h"
#include "gemm_split.h"
#include "internal.h"
#include "jacobi_ops.h"
#include "wave_ops.h"

namespace mps {

namespace {

inline int cdiv(long long a, long long b) { return (int)((a + b - 1) / b); }

}  // namespace

// =================================================================== state

__global__ void init_product_kernel(double2* const* sites, double* const* lam, const uint8_t* bits,
                                    int n) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n) {
    const int b = bits[q] ? 1 : 0;
    sites[q][0] = make_double2(b == 0 ? 1.0 : 0.0, 0.0);
    sites[q][1] = make_double2(b == 1 ? 1.0 : 0.0, 0.0);
  }
  if (q <= n) lam[q][0] = 1.0;
}

hipError_t launch_init_product(double2* const* sites, double* const* lam0, const uint8_t* bits,
                               int n, hipStream_t s) {
  hipLaunchKernelGGL(init_product_kernel, dim3(cdiv(n + 1, 256)), dim3(256), 0, s, sites, lam0,
                     bits, n);
  return hipGetLastError();
}

// Eq. (1q): B^s <- sum_s' Q_{ss'} B^{s'}; count = Dl * Dr elements per physical index.
__global__ void gate1q_kernel(double2* b, const double2* u, int count) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const double2 x0 = b[i], x1 = b[count + i];
  const double2 u00 = u[0], u01 = u[1], u10 = u[2], u11 = u[3];
  const double2 a = cmul(u00, x0), bb = cmul(u01, x1), c = cmul(u10, x0), d = cmul(u11, x1);
  b[i] = make_double2(a.x + bb.x, a.y + bb.y);
  b[count + i] = make_double2(c.x + d.x, c.y + d.y);
}

hipError_t launch_gate1q(double2* b, const double2* u, int count, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(gate1q_kernel, dim3(cdiv(count, 256)), dim3(256), 0, s, b, u, count);
  return hipGetLastError();
}

// =================================================================== Eq. (C)

struct ThetaP {
  using T = double;
  using Ctx = ThetaItem;
  static constexpr bool A_CONTIG_K = true, B_CONTIG_N = true, REAL_ONLY = false;
  const ThetaItem* items;
  __device__ Ctx context(int i) const { return items[i]; }
  __device__ static void dims(const Ctx& c, int& M, int& N, int& K) {
    M = 2 * c.dl;
    N = 2 * c.dr;
    K = c.dm;
  }
  using RowA = const double2*;
  using ColB = const double2*;
  __device__ static RowA rowA(const Ctx& c, int i) { return c.bl + (size_t)i * c.dm; }
  __device__ static ColB colB(const Ctx& c, int j) {
    const int s = j >= c.dr;
    return c.br + (size_t)s * c.dm * c.dr + (j - s * c.dr);
  }
  __device__ static double2 loadA(const Ctx&, RowA r, int, int k) { return r[k]; }
  __device__ static double2 loadB(const Ctx& c, ColB b, int k, int) { return b[(size_t)k * c.dr]; }
  __device__ static void store(const Ctx& c, int i, int j, double re, double im) {
    c.theta[(size_t)i * (2 * c.dr) + j] = make_double2(re, im);
  }
};

hipError_t launch_theta(const ThetaItem* items_dev, int items, int max_rows, int max_cols,
                        hipStream_t s) {
  ThetaP p{items_dev};
  return launch_cgemm<64, 64, 16>(p, items, max_rows, max_cols, s);
}

// C^{t1 t2}_{l r} = sum_{s1 s2} Q[(t1 t2),(s1 s2)] Theta[(s1,l),(s2,r)]  (Eq. C)
// W = lambda_l C                                                       (Eq. C~)
// One thread per (l, r); ||W||_F^2 accumulated per item.
__global__ __launch_bounds__(256) void mix_kernel(const MixItem* items, int per_item_blocks) {
  const int item = blockIdx.x / per_item_blocks;
  const int blk = blockIdx.x - item * per_item_blocks;
  const MixItem it = items[item];
  const int dl = it.dl, dr = it.dr;
  const int idx = blk * 256 + threadIdx.x;
  double local = 0.0;
  if (idx < dl * dr) {
    const int l = idx / dr, r = idx - (idx / dr) * dr;
    const size_t ld = 2 * (size_t)dr;
    double2 th[4];
#pragma unroll
    for (int s1 = 0; s1 < 2; ++s1)
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2) th[s1 * 2 + s2] = it.c[(size_t)(s1 * dl + l) * ld + s2 * dr + r];
    const double lam = it.lam[l];
#pragma unroll
    for (int t1 = 0; t1 < 2; ++t1)
#pragma unroll
      for (int t2 = 0; t2 < 2; ++t2) {
        double2 acc = make_double2(0.0, 0.0);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const double2 v = cmul(it.q[(t1 * 2 + t2) * 4 + k], th[k]);
          acc.x += v.x;
          acc.y += v.y;
        }
        const size_t o = (size_t)(t1 * dl + l) * ld + t2 * dr + r;
        it.c[o] = acc;
        const double2 wv = make_double2(lam * acc.x, lam * acc.y);
        it.w[o] = wv;
        local += wv.x * wv.x + wv.y * wv.y;
      }
  }
  local = wave_sum(local);
  __shared__ double part[4];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = local;
  __syncthreads();
  if (threadIdx.x == 0) atomicAdd(it.fro2, part[0] + part[1] + part[2] + part[3]);
}

hipError_t launch_mix(const MixItem* items_dev, int items, int max_dldr, hipStream_t s) {
  if (items <= 0) return hipSuccess;
  const int per = cdiv(max_dldr, 256);
  hipLaunchKernelGGL(mix_kernel, dim3(items * per), dim3(256), 0, s, items_dev, per);
  return hipGetLastError();
}

// =================================================================== Algorithm 1

// Rotate local vectors i and j (one wave): b_ii, b_jj, b_ij by wave
// reductions, then, if |b_ij| > eps sqrt(b_ii b_jj) and |b_ij| > floor,
//   tau = (b_ii - b_jj) / (2|b_ij|), t = sign(tau) / (|tau| + sqrt(1 + tau^2)),
//   c = 1/sqrt(1+t^2), s = t c, e = b_ij / |b_ij|,
//   a_i <- c a_i + s conj(e) a_j,   a_j <- c a_j - s e a_i.
__device__ __forceinline__ bool jacobi_pair(double2* xi, double2* xj, int m, int lane, double eps,
                                            double floor) {
  double bii = 0.0, bjj = 0.0, br = 0.0, bi = 0.0;
  for (int e = lane; e < m; e += 64) {
    const double2 a = xi[e], b = xj[e];
    bii += a.x * a.x + a.y * a.y;
    bjj += b.x * b.x + b.y * b.y;
    br += a.x * b.x + a.y * b.y;
    bi += a.x * b.y - a.y * b.x;
  }
  bii = wave_sum(bii);
  bjj = wave_sum(bjj);
  br = wave_sum(br);
  bi = wave_sum(bi);
  const double mag = sqrt(br * br + bi * bi);
  if (!(mag > floor) || !(mag > eps * sqrt(bii * bjj))) return false;
  const double tau = (bii - bjj) / (2.0 * mag);
  const double at = fabs(tau);
  const double sg = tau >= 0.0 ? 1.0 : -1.0;
  const double t = at > 1e100 ? sg * (0.5 / at) : sg / (at + sqrt(1.0 + tau * tau));
  const double c = 1.0 / sqrt(1.0 + t * t);
  const double s = t * c;
  const double er = br / mag, ei = bi / mag;
  for (int e = lane; e < m; e += 64) {
    const double2 a = xi[e], b = xj[e];
    // conj(e) b and e a
    const double cbr = er * b.x + ei * b.y, cbi = er * b.y - ei * b.x;
    const double ear = er * a.x - ei * a.y, eai = er * a.y + ei * a.x;
    xi[e] = make_double2(c * a.x + s * cbr, c * a.y + s * cbi);
    xj[e] = make_double2(c * b.x - s * ear, c * b.y - s * eai);
  }
  return true;
}

// One sweep over all pairs of the nloc local vectors in round-robin order
// (nloc - 1 rounds of nloc/2 disjoint pairs, one pair per wave at a time).
// gidx gives each local vector's global index (-1 = absent); pairs are
// oriented so the lower global index plays the role of i.
__device__ int jacobi_local_sweep(double2* sm, const int* gidx, int nloc, int m, double eps,
                                  double floor, int* s_rot) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int nwaves = blockDim.x >> 6;
  if (threadIdx.x == 0) *s_rot = 0;
  __syncthreads();
  for (int ir = 0; ir < nloc - 1; ++ir) {
    for (int pp = wave; pp < nloc / 2; pp += nwaves) {
      int i = (pp == 0) ? 0 : 1 + ((pp - 1 + ir) % (nloc - 1));
      int j = 1 + ((nloc - 2 - pp + ir) % (nloc - 1));
      const int gi = gidx[i], gj = gidx[j];
      if (gi < 0 || gj < 0) continue;
      if (gi > gj) {
        const int tmp = i;
        i = j;
        j = tmp;
      }
      if (jacobi_pair(sm + (size_t)i * m, sm + (size_t)j * m, m, lane, eps, floor) && lane == 0)
        atomicAdd(s_rot, 1);
    }
    __syncthreads();
  }
  return *s_rot;
}

// Block mode: one workgroup per block pair of round `round`; the pair's
// 2*wblk vectors are staged in LDS, swept once, and written back.  Each block
// is a contiguous run of vectors, so staging is two flat, coalesced copies.
__global__ __launch_bounds__(512) void jacobi_block_kernel(const JacItem* items, int max_pairs,
                                                           int round, int sweep, double eps_scale) {
  extern __shared__ double2 sm[];
  __shared__ int gidx[256];
  __shared__ int s_rot;
  const int item = blockIdx.x / max_pairs;
  const int p = blockIdx.x - item * max_pairs;
  const JacItem it = items[item];
  const int nb = it.nb;
  if (p >= nb / 2 || round >= nb - 1) return;
  if (sweep > 0 && it.rot[(sweep - 1) * it.rot_stride] == 0) return;  // converged
  const int w = it.wblk, m = it.m, n = it.n;
  const int bp = (p == 0) ? 0 : 1 + ((p - 1 + round) % (nb - 1));
  const int bq = 1 + ((nb - 2 - p + round) % (nb - 1));
  const int nloc = 2 * w;
  for (int lv = threadIdx.x; lv < nloc; lv += blockDim.x) {
    const int g = lv < w ? bp * w + lv : bq * w + (lv - w);
    gidx[lv] = g < n ? g : -1;
  }
  const int vp = max(0, min(w, n - bp * w)), vq = max(0, min(w, n - bq * w));
  const size_t cp = (size_t)vp * m, cq = (size_t)vq * m, wm = (size_t)w * m;
  const double2* srcp = it.w + (size_t)bp * w * m;
  const double2* srcq = it.w + (size_t)bq * w * m;
#pragma unroll 4
  for (size_t i = threadIdx.x; i < wm; i += 512) sm[i] = i < cp ? srcp[i] : make_double2(0.0, 0.0);
#pragma unroll 4
  for (size_t i = threadIdx.x; i < wm; i += 512) sm[wm + i] = i < cq ? srcq[i] : make_double2(0.0, 0.0);
  __syncthreads();
  const double eps = eps_scale * (double)m;
  const double floor = eps * eps * (*it.fro2);
  const int rot = jacobi_local_sweep(sm, gidx, nloc, m, eps, floor, &s_rot);
  if (rot > 0) {
    double2* dstp = it.w + (size_t)bp * w * m;
    double2* dstq = it.w + (size_t)bq * w * m;
#pragma unroll 4
    for (size_t i = threadIdx.x; i < cp; i += 512) dstp[i] = sm[i];
#pragma unroll 4
    for (size_t i = threadIdx.x; i < cq; i += 512) dstq[i] = sm[wm + i];
    if (threadIdx.x == 0) atomicAdd(&it.rot[sweep * it.rot_stride], rot);
  }
}

// ---------------------------------------------------------------------------
// Register-resident block Jacobi on blocks of JW = 8 vectors; each lane keeps
// E elements (e = lane + 64 k) of the vectors its wave holds, so dot products
// and rotations never touch LDS.  A sweep is one launch for the 28 pairs
// inside every block (circle method, both vectors of a wave move each inner
// round), then one launch per outer round of the block round-robin, each
// pairing every block with exactly one other and taking the 64 cross pairs
// of the two (resident vectors stay, travellers move one wave along per
// inner round).  Over one sweep every pair of the matrix is visited once.
constexpr int JW = 8;

template <int E>
struct RegVec {
  double2 v[E];
};

// Every lane loads (unconditionally, from inside the row: indices past the
// row end are clamped to its last element; src is always a row of the
// matrix) and zeroes what lies outside the row or belongs to a padding row,
// so the loads need no branches.
template <int E>
__device__ __forceinline__ void rv_load(RegVec<E>& r, const double2* src, int valid, int m, int lane) {
  const gdvec2* g = (const gdvec2*)src;
#pragma unroll
  for (int k = 0; k < E; ++k) {
    const int e = lane + 64 * k;
    const dvec2 v = g[e < m ? e : m - 1];
    const bool keep = valid && e < m;
    r.v[k] = make_double2(keep ? v.x : 0.0, keep ? v.y : 0.0);
  }
}

template <int E>
__device__ __forceinline__ void rv_store(const RegVec<E>& r, double2* dst, int m, int lane) {
  gdvec2* g = (gdvec2*)dst;
#pragma unroll
  for (int k = 0; k < E; ++k) {
    const int e = lane + 64 * k;
    if (e < m) g[e] = dvec2{r.v[k].x, r.v[k].y};
  }
}

template <int E>
__device__ __forceinline__ void rv_to_lds(const RegVec<E>& r, double2* slot, int lane) {
#pragma unroll
  for (int k = 0; k < E; ++k) slot[64 * k + lane] = r.v[k];
}

template <int E>
__device__ __forceinline__ void rv_from_lds(RegVec<E>& r, const double2* slot, int lane) {
#pragma unroll
  for (int k = 0; k < E; ++k) r.v[k] = slot[64 * k + lane];
}

template <int E>
__device__ __forceinline__ double rv_norm2(const RegVec<E>& r) {
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < E; ++k) s = norm_acc(r.v[k], s);
  return wave_sum(s);
}

// Algorithm 1's pair step on register vectors x (as a_i) and y (as a_j) with
// their squared norms nx and ny, which move with the rotation: only x^+y is
// reduced.  (Exchanging the parts of a_i and a_j gives the same rotation.)
template <int E>
__device__ __forceinline__ bool jacobi_pair_tracked(RegVec<E>& x, double& nx, RegVec<E>& y, double& ny,
                                                    double eps, double floor, int lane) {
  double v[2];
  pair_partials_xy<E>(x.v, y.v, v[0], v[1]);
  wave_sum_scalar<2>(v, lane);
  if (!pair_needs_rot(nx, ny, v[0], v[1], eps, floor)) return false;
  Rot rt;
  double dn;
  pair_rot_coeffs(nx, ny, v[0], v[1], rt, &dn);
  rt.c = wave_uniform(rt.c);
  rt.ar = wave_uniform(rt.ar);
  rt.ai = wave_uniform(rt.ai);
  rt.br = -rt.ar;
  rt.bi = rt.ai;
  pair_apply<E>(x.v, y.v, rt);
  nx += dn;
  ny -= dn;
  return true;
}

// Common prologue of the register kernels: which block pair this workgroup
// owns, or false if it has nothing to do (padding pair, converged item).
struct RegCtx {
  JacItem it;
  int bp, bq;
  double eps, floor;
};

__device__ __forceinline__ bool reg_prologue(const JacItem* items, int max_pairs, int round,
                                             int sweep, double eps_scale, RegCtx& c) {
  const int item = blockIdx.x / max_pairs;
  const int p = blockIdx.x - item * max_pairs;
  c.it = items[item];
  const int nb = c.it.nb;
  if (p >= nb / 2 || round >= nb - 1) return false;
  if (sweep > 0 && c.it.rot[(sweep - 1) * c.it.rot_stride] == 0) return false;  // converged
  c.bp = (p == 0) ? 0 : 1 + ((p - 1 + round) % (nb - 1));
  c.bq = 1 + ((nb - 2 - p + round) % (nb - 1));
  c.eps = eps_scale * (double)c.it.m;
  c.floor = c.eps * c.eps * (*c.it.fro2);
  return true;
}

// Circle method over the 2W rows that W waves hold (wave w: positions w and
// 2W - 1 - w): every pair of them is visited once in 2W - 1 steps; after
// each step positions 1..2W-1 advance by one through 2 x W LDS slots
// (position 0 fixed), in C chunks of E / C elements per lane so that the
// slots take 2 W 64 (E / C) elements.  gx, gy (global indices, -1 padding)
// and the squared norms follow the rows.
template <int E, int W, int C>
__device__ __forceinline__ int circle_pairs(RegVec<E>& x, int& gx, RegVec<E>& y, int& gy, double2* slots,
                                            int* g_top, int* g_bot, double* n_top, double* n_bot, double eps,
                                            double floor, int lane, int wv) {
  static_assert(E % C == 0, "chunks must divide the elements per lane");
  constexpr int EC = E / C;
  double2* top = slots;
  double2* bot = slots + (size_t)W * 64 * EC;
  int rot = 0;
  double sx = rv_norm2<E>(x), sy = rv_norm2<E>(y);
  for (int t = 0; t < 2 * W - 1; ++t) {
    rot += jacobi_pair_tracked<E>(x, sx, y, sy, eps, floor, lane);
    int nx = gx, ny = gy;
#pragma unroll
    for (int c = 0; c < C; ++c) {
#pragma unroll
      for (int k = 0; k < EC; ++k) {
        top[((size_t)wv * EC + k) * 64 + lane] = x.v[c * EC + k];
        bot[((size_t)wv * EC + k) * 64 + lane] = y.v[c * EC + k];
      }
      if (c == 0 && lane == 0) {
        g_top[wv] = gx;
        g_bot[wv] = gy;
        n_top[wv] = sx;
        n_bot[wv] = sy;
      }
      __syncthreads();
      // new pos j+1 <- old pos j for j = 1..2W-2, new pos 1 <- old pos 2W-1, pos 0 fixed
      const double2* px = wv >= 2 ? top + (size_t)(wv - 1) * EC * 64 : (wv == 1 ? bot : nullptr);
      const double2* py = wv <= W - 2 ? bot + (size_t)(wv + 1) * EC * 64 : top + (size_t)(W - 1) * EC * 64;
      if (px) {
#pragma unroll
        for (int k = 0; k < EC; ++k) x.v[c * EC + k] = px[(size_t)k * 64 + lane];
      }
#pragma unroll
      for (int k = 0; k < EC; ++k) y.v[c * EC + k] = py[(size_t)k * 64 + lane];
      if (c == 0) {
        if (wv >= 1) {
          nx = wv >= 2 ? g_top[wv - 1] : g_bot[0];
          sx = wv >= 2 ? n_top[wv - 1] : n_bot[0];
        }
        ny = wv <= W - 2 ? g_bot[wv + 1] : g_top[W - 1];
        sy = wv <= W - 2 ? n_bot[wv + 1] : n_top[W - 1];
      }
      __syncthreads();
    }
    gx = nx;
    gy = ny;
  }
  return rot;
}

// The 28 pairs inside each block of 8 rows, one 4-wave workgroup per block
// (rows b*8 + w and b*8 + 7 - w on wave w), for every block of every item.
// Run before outer round 0 of a sweep, whose cross pairs the cross kernel
// then takes: over the sweep every pair of the matrix is visited once.  The
// rows move through LDS in two halves (32 KB at E = 8), so that LDS allows
// as many resident workgroups as the registers do.
constexpr int IW = JW / 2;
template <int E>
constexpr int intra_chunks() { return E >= 2 ? 2 : 1; }

template <int E>
__global__ __launch_bounds__(IW * 64) void jacobi_reg_intra_kernel(const JacItem* items, int max_blocks,
                                                                   int sweep, double eps_scale) {
  extern __shared__ double2 slots[];  // 2 * IW slots of 64 * E / intra_chunks<E>() elements
  __shared__ int s_rot;
  __shared__ int g_top[IW], g_bot[IW];
  __shared__ double n_top[IW], n_bot[IW];
  const int item = blockIdx.x / max_blocks;
  const int b = blockIdx.x - item * max_blocks;
  const JacItem it = items[item];
  if (b >= it.nb) return;
  if (sweep > 0 && it.rot[(sweep - 1) * it.rot_stride] == 0) return;  // converged
  const int m = it.m, n = it.n;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (threadIdx.x == 0) s_rot = 0;
  const double eps = eps_scale * (double)m;
  const double floor = eps * eps * (*it.fro2);
  RegVec<E> x, y;
  int gx = b * JW + wv, gy = b * JW + (JW - 1 - wv);
  gx = gx < n ? gx : -1;
  gy = gy < n ? gy : -1;
  rv_load<E>(x, it.w + (size_t)max(gx, 0) * m, gx >= 0, m, lane);
  rv_load<E>(y, it.w + (size_t)max(gy, 0) * m, gy >= 0, m, lane);
  const int rot = circle_pairs<E, IW, intra_chunks<E>()>(x, gx, y, gy, slots, g_top, g_bot, n_top, n_bot, eps, floor,
                                                            lane, wv);
  if (lane == 0 && rot) atomicAdd(&s_rot, rot);
  __syncthreads();
  if (s_rot > 0) {
    if (gx >= 0) rv_store<E>(x, it.w + (size_t)gx * m, m, lane);
    if (gy >= 0) rv_store<E>(y, it.w + (size_t)gy * m, m, lane);
    if (threadIdx.x == 0) atomicAdd(&it.rot[sweep * it.rot_stride], s_rot);
  }
}

// Two disjoint pairs (x0, y0), (x1, y1) with their squared norms tracked:
// only x^+y is reduced (4 partial sums, reduce-scattered over lane bits 3
// and 2, then full sums over bits 1, 0, 4, 5), so lane l holds component
// (l >> 3) & 1 (Re, Im) of pair (l >> 2) & 1; the other component comes by a
// row rotation, the rotation is computed lane-parallel and the norms move by
// +-t |b_ij| (Algorithm 1 recomputes them; the caller does so at every
// launch, so at most a few updates accumulate).
template <int E>
__device__ __forceinline__ int rot2n(RegVec<E>& x0, RegVec<E>& y0, double& nx0, double& ny0,
                                     RegVec<E>& x1, RegVec<E>& y1, double& nx1, double& ny1,
                                     double eps, double floor, int lane) {
  double v[4];  // v[2c + i]: component c (0 Re, 1 Im) of pair i
  pair_partials_xy<E>(x0.v, y0.v, v[0], v[2]);
  pair_partials_xy<E>(x1.v, y1.v, v[1], v[3]);
  double v2[2], x;
  {
    const bool hi = (lane >> 3) & 1;
#pragma unroll
    for (int j = 0; j < 2; ++j)
      v2[j] = (hi ? v[2 + j] : v[j]) + dpp_mov<0x140>(hi ? v[j] : v[2 + j]);
  }
  {
    const bool hi = (lane >> 2) & 1;
    x = (hi ? v2[1] : v2[0]) + dpp_mov<0x141>(hi ? v2[0] : v2[1]);
  }
  x += dpp_mov<0x4E>(x);
  x += dpp_mov<0xB1>(x);
  x = add_xor32(add_xor16(x));
  const double other = dpp_mov<0x128>(x);  // row_ror:8, the lane with the other component
  const bool im_lane = (lane >> 3) & 1;
  const bool p1 = (lane >> 2) & 1;
  const double bxx = p1 ? nx1 : nx0, byy = p1 ? ny1 : ny0;
  const double br = im_lane ? other : x, bi = im_lane ? x : other;
  const uint64_t act = __ballot(pair_needs_rot(bxx, byy, br, bi, eps, floor));
  if (!(act & 17ull)) return 0;  // neither pair rotates: skip the rotation formula
  Rot mine;
  double dn;
  pair_rot_coeffs(bxx, byy, br, bi, mine, &dn);
  int rot = 0;
  // pair i is held (Re component) by lane 4 i
  if (act & 1ull) {
    Rot rt{readlane_d(mine.c, 0), readlane_d(mine.ar, 0), readlane_d(mine.ai, 0), 0.0, 0.0};
    rt.br = -rt.ar;
    rt.bi = rt.ai;
    const double d = readlane_d(dn, 0);
    pair_apply<E>(x0.v, y0.v, rt);
    nx0 += d;
    ny0 -= d;
    ++rot;
  }
  if (act & 16ull) {
    Rot rt{readlane_d(mine.c, 4), readlane_d(mine.ar, 4), readlane_d(mine.ai, 4), 0.0, 0.0};
    rt.br = -rt.ar;
    rt.bi = rt.ai;
    const double d = readlane_d(dn, 4);
    pair_apply<E>(x1.v, y1.v, rt);
    nx1 += d;
    ny1 -= d;
    ++rot;
  }
  return rot;
}

// Every outer round: the 64 cross pairs of blocks bp and bq on CW = 4 waves.
// Wave w keeps resident rows bp*8 + 2w, 2w + 1 and holds two travellers from
// block bq, which move one wave along per step through LDS (4 steps) with
// their squared norms; each step is two sub-steps of two disjoint pairs.
constexpr int CW = 4;

template <int E>
__global__ __launch_bounds__(CW * 64, 2) void jacobi_reg_cross_kernel(const JacItem* items, int max_pairs,
                                                                      int round, int sweep,
                                                                      double eps_scale) {
  extern __shared__ double2 slots[];  // CW slots of two travellers (2 x 64 E elements)
  __shared__ double s_tn[CW][2];      // the travellers' squared norms
  __shared__ int s_rot;
  RegCtx c;
  if (!reg_prologue(items, max_pairs, round, sweep, eps_scale, c)) return;
  const int m = c.it.m, n = c.it.n;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (threadIdx.x == 0) s_rot = 0;
  RegVec<E> r0, r1, t0, t1;
  const int g0 = c.bp * JW + 2 * wv, g1 = g0 + 1;
  rv_load<E>(r0, c.it.w + (size_t)min(g0, n - 1) * m, g0 < n, m, lane);
  rv_load<E>(r1, c.it.w + (size_t)min(g1, n - 1) * m, g1 < n, m, lane);
  int src = wv;  // home wave of the travellers held
  {
    const int h0 = c.bq * JW + 2 * src, h1 = h0 + 1;
    rv_load<E>(t0, c.it.w + (size_t)min(h0, n - 1) * m, h0 < n, m, lane);
    rv_load<E>(t1, c.it.w + (size_t)min(h1, n - 1) * m, h1 < n, m, lane);
  }
  double nr0 = rv_norm2<E>(r0), nr1 = rv_norm2<E>(r1), nt0 = rv_norm2<E>(t0), nt1 = rv_norm2<E>(t1);
  int rot = 0;
  for (int st = 0; st < CW; ++st) {
    rot += rot2n<E>(r0, t0, nr0, nt0, r1, t1, nr1, nt1, c.eps, c.floor, lane);
    rot += rot2n<E>(r0, t1, nr0, nt1, r1, t0, nr1, nt0, c.eps, c.floor, lane);
    if (st == CW - 1) break;
    double2* mine = slots + (size_t)wv * 2 * 64 * E;
    rv_to_lds<E>(t0, mine, lane);
    rv_to_lds<E>(t1, mine + 64 * E, lane);
    if (lane == 0) {
      s_tn[wv][0] = nt0;
      s_tn[wv][1] = nt1;
    }
    __syncthreads();
    const int from = (wv + CW - 1) % CW;
    const double2* prev = slots + (size_t)from * 2 * 64 * E;
    rv_from_lds<E>(t0, prev, lane);
    rv_from_lds<E>(t1, prev + 64 * E, lane);
    nt0 = s_tn[from][0];
    nt1 = s_tn[from][1];
    src = (src + CW - 1) % CW;
    __syncthreads();
  }
  if (lane == 0 && rot) atomicAdd(&s_rot, rot);
  __syncthreads();
  if (s_rot > 0) {
    const int h0 = c.bq * JW + 2 * src, h1 = h0 + 1;
    if (g0 < n) rv_store<E>(r0, c.it.w + (size_t)g0 * m, m, lane);
    if (g1 < n) rv_store<E>(r1, c.it.w + (size_t)g1 * m, m, lane);
    if (h0 < n) rv_store<E>(t0, c.it.w + (size_t)h0 * m, m, lane);
    if (h1 < n) rv_store<E>(t1, c.it.w + (size_t)h1 * m, m, lane);
    if (threadIdx.x == 0) atomicAdd(&c.it.rot[sweep * c.it.rot_stride], s_rot);
  }
}

template <int E>
hipError_t launch_reg_e(const JacItem* items_dev, int items, int max_pairs, int round, int sweep,
                        double eps_scale, hipStream_t s) {
  if (round == 0) {  // in-block pairs of every block first (nb = 2 * pairs blocks per item)
    hipLaunchKernelGGL(jacobi_reg_intra_kernel<E>, dim3(items * 2 * max_pairs), dim3(IW * 64),
                       2 * IW * 64 * (E / intra_chunks<E>()) * sizeof(double2), s, items_dev, 2 * max_pairs,
                       sweep, eps_scale);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(jacobi_reg_cross_kernel<E>, dim3(items * max_pairs), dim3(CW * 64),
                     CW * 2 * 64 * E * sizeof(double2), s, items_dev, max_pairs, round, sweep, eps_scale);
  return hipGetLastError();
}

// Rows of 513..1024 elements (E = 16, 64 registers per row and lane): a wave
// keeps one resident row of block bp in registers and takes its partners
// from LDS, where the eight rows of block bq sit (128 KB).  Cross rounds are
// eight steps; at step st wave w pairs its resident row with LDS row
// (w + st) % 8, a permutation, so no row is touched twice in a step.  Outer
// round 0 first sweeps the 28 pairs inside each block (block bp, then bq, in
// LDS, circle method, four waves with both rows in registers), then the 64
// cross pairs, so that every pair is visited once per outer sweep as with
// the shorter rows.
template <int E, int NW>
__device__ __forceinline__ int lds_intra_block(double2* lds, double* nrm, double eps, double floor, int wv,
                                               int lane) {
  int rot = 0;
  for (int t = 0; t < NW - 1; ++t) {
    if (wv < NW / 2) {
      auto pos = [&](int k) { return k == 0 ? 0 : 1 + (k - 1 + t) % (NW - 1); };
      const int a = pos(wv), bb = pos(NW - 1 - wv);
      RegVec<E> x, y;
      rv_from_lds<E>(x, lds + (size_t)a * 64 * E, lane);
      rv_from_lds<E>(y, lds + (size_t)bb * 64 * E, lane);
      double nx = nrm[a], ny = nrm[bb];
      if (jacobi_pair_tracked<E>(x, nx, y, ny, eps, floor, lane)) {
        rv_to_lds<E>(x, lds + (size_t)a * 64 * E, lane);
        rv_to_lds<E>(y, lds + (size_t)bb * 64 * E, lane);
        if (lane == 0) {
          nrm[a] = nx;
          nrm[bb] = ny;
        }
        ++rot;
      }
    }
    __syncthreads();
  }
  return rot;
}

// Blocks of NW rows on NW waves: each wave keeps one resident row of block bp
// in registers and takes its partners from LDS, where the NW rows of block bq
// sit (NW * 64 E complex values).  Cross rounds are NW steps; at step st wave
// w pairs its resident row with LDS row (w + st) % NW, a permutation, so no
// row is touched twice in a step.  Outer round 0 first sweeps the pairs
// inside each block (block bp, then bq, in LDS, circle method, NW / 2 waves
// with both rows in registers), then the cross pairs, so that every pair is
// visited once per outer sweep.  Used with E = 16 (513..1024-long rows) and
// NW = 8, the block size of the other register kernels.
template <int E, int NW>
__global__ __launch_bounds__(NW * 64, 1) void jacobi_reg_lds_kernel(const JacItem* items, int max_pairs,
                                                                    int round, int sweep, double eps_scale) {
  extern __shared__ double2 lds[];  // NW rows of 64 E elements
  __shared__ int s_rot;
  __shared__ double s_nrm[NW];  // their squared norms, fresh at every launch, then tracked
  RegCtx c;
  if (!reg_prologue(items, max_pairs, round, sweep, eps_scale, c)) return;
  const int m = c.it.m, n = c.it.n;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // the block pair in units of NW rows (the prologue's indices are in units of the item's blocks)
  const int bp = c.bp, bq = c.bq;
  if (threadIdx.x == 0) s_rot = 0;
  int rot = 0;
  auto block_to_lds = [&](int b) {
    const int g = b * NW + wv;
    RegVec<E> v;
    rv_load<E>(v, c.it.w + (size_t)min(g, n - 1) * m, g < n, m, lane);
    rv_to_lds<E>(v, lds + (size_t)wv * 64 * E, lane);
    const double nn = rv_norm2<E>(v);
    if (lane == 0) s_nrm[wv] = nn;
  };
  const int gx = bp * NW + wv;
  if (round == 0) {
    // block bp's own pairs in LDS; its rows go back to memory (each lane
    // rewrites and later rereads only its own elements) so that no resident
    // row is held while the other block's pairs take two rows per wave
    block_to_lds(bp);
    __syncthreads();
    rot += lds_intra_block<E, NW>(lds, s_nrm, c.eps, c.floor, wv, lane);
    if (gx < n)
      for (int k = 0; k < E; ++k) {
        const int e = lane + 64 * k;
        if (e < m) c.it.w[(size_t)gx * m + e] = lds[(size_t)wv * 64 * E + 64 * k + lane];
      }
    __syncthreads();  // every row is read before block bq overwrites LDS
  }
  block_to_lds(bq);
  __syncthreads();
  if (round == 0) rot += lds_intra_block<E, NW>(lds, s_nrm, c.eps, c.floor, wv, lane);
  RegVec<E> x;  // resident row wv of block bp
  rv_load<E>(x, c.it.w + (size_t)min(gx, n - 1) * m, gx < n, m, lane);
  double nx = rv_norm2<E>(x);
  for (int st = 0; st < NW; ++st) {
    const int j = (wv + st) % NW;
    RegVec<E> y;
    rv_from_lds<E>(y, lds + (size_t)j * 64 * E, lane);
    double ny = s_nrm[j];
    if (jacobi_pair_tracked<E>(x, nx, y, ny, c.eps, c.floor, lane)) {
      rv_to_lds<E>(y, lds + (size_t)j * 64 * E, lane);
      if (lane == 0) s_nrm[j] = ny;
      ++rot;
    }
    __syncthreads();
  }
  if (lane == 0 && rot) atomicAdd(&s_rot, rot);
  __syncthreads();
  if (s_rot > 0) {
    if (gx < n) rv_store<E>(x, c.it.w + (size_t)gx * m, m, lane);
    const int gq = bq * NW + wv;
    if (gq < n)
      for (int k = 0; k < E; ++k) {
        const int e = lane + 64 * k;
        if (e < m) c.it.w[(size_t)gq * m + e] = lds[(size_t)wv * 64 * E + 64 * k + lane];
      }
    if (threadIdx.x == 0) atomicAdd(&c.it.rot[sweep * c.it.rot_stride], s_rot);
  }
}

constexpr size_t kWideLds = (size_t)8 * 64 * 16 * sizeof(double2);  // 128 KB

// Rows of 513..1024 elements: E = 16, 8-row blocks.  (The same design with
// E = 8 and 16-row blocks, half the rounds of the 8-row register blocks, was
// slower than jacobi_reg_cross_kernel on 512-long rows: 159 against 101 ms
// per saturated 50-qubit D = 256 layer.)
hipError_t launch_jacobi_wide(const JacItem* items_dev, int items, int max_pairs, int round, int sweep,
                              double eps_scale, hipStream_t s) {
  if (items <= 0 || max_pairs <= 0) return hipSuccess;
  hipLaunchKernelGGL((jacobi_reg_lds_kernel<16, 8>), dim3(items * max_pairs), dim3(8 * 64), kWideLds, s,
                     items_dev, max_pairs, round, sweep, eps_scale);
  return hipGetLastError();
}

hipError_t launch_jacobi_reg(const JacItem* items_dev, int items, int max_pairs, int round,
                             int sweep, double eps_scale, int max_m, hipStream_t s) {
  if (items <= 0 || max_pairs <= 0) return hipSuccess;
  if (max_m <= 64) return launch_reg_e<1>(items_dev, items, max_pairs, round, sweep, eps_scale, s);
  if (max_m <= 128) return launch_reg_e<2>(items_dev, items, max_pairs, round, sweep, eps_scale, s);
  if (max_m <= 256) return launch_reg_e<4>(items_dev, items, max_pairs, round, sweep, eps_scale, s);
  if (max_m <= 512) return launch_reg_e<8>(items_dev, items, max_pairs, round, sweep, eps_scale, s);
  return hipErrorInvalidValue;
}

// Single mode: the whole matrix fits in LDS; sweep until a sweep performs no
// rotation or max_sweeps is reached.
__global__ __launch_bounds__(512) void jacobi_single_kernel(const JacItem* items, int max_sweeps,
                                                            double eps_scale) {
  extern __shared__ double2 sm[];
  __shared__ int gidx[1024];
  __shared__ int s_rot;
  const JacItem it = items[blockIdx.x];
  const int n = it.n, m = it.m;
  const int nloc = (n + 1) & ~1;
  for (int lv = threadIdx.x; lv < nloc; lv += blockDim.x) gidx[lv] = lv < n ? lv : -1;
  for (int idx = threadIdx.x; idx < n * m; idx += blockDim.x) sm[idx] = it.w[idx];
  __syncthreads();
  const double eps = eps_scale * (double)m;
  const double floor = eps * eps * (*it.fro2);
  int done = -max_sweeps;
  int any = 0;
  for (int sw = 0; sw < max_sweeps; ++sw) {
    const int rot = jacobi_local_sweep(sm, gidx, nloc, m, eps, floor, &s_rot);
    __syncthreads();
    any += rot;
    if (rot == 0) {
      done = sw + 1;
      break;
    }
  }
  if (any > 0)
    for (int idx = threadIdx.x; idx < n * m; idx += blockDim.x) it.w[idx] = sm[idx];
  if (threadIdx.x == 0) *it.sweeps_done = done;
}

hipError_t configure_jacobi_lds(size_t bytes) {
  const void* fns[] = {(const void*)jacobi_block_kernel, (const void*)jacobi_single_kernel,
                       (const void*)jacobi_reg_intra_kernel<1>, (const void*)jacobi_reg_intra_kernel<2>,
                       (const void*)jacobi_reg_intra_kernel<4>, (const void*)jacobi_reg_intra_kernel<8>,
                       (const void*)jacobi_reg_cross_kernel<1>, (const void*)jacobi_reg_cross_kernel<2>,
                       (const void*)jacobi_reg_cross_kernel<4>, (const void*)jacobi_reg_cross_kernel<8>};
  for (const void* f : fns) {
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess) return e;
  }
  if (bytes >= kWideLds) {
    const void* lf[] = {(const void*)jacobi_reg_lds_kernel<16, 8>};
    for (const void* f : lf) {
      hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kWideLds);
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

hipError_t launch_jacobi_block(const JacItem* items_dev, int items, int max_pairs, int round,
                               int sweep, double eps_scale, size_t lds_bytes, hipStream_t s) {
  if (items <= 0 || max_pairs <= 0) return hipSuccess;
  hipLaunchKernelGGL(jacobi_block_kernel, dim3(items * max_pairs), dim3(512), lds_bytes, s,
                     items_dev, max_pairs, round, sweep, eps_scale);
  return hipGetLastError();
}

hipError_t launch_jacobi_single(const JacItem* items_dev, int items, int max_sweeps,
                                double eps_scale, size_t lds_bytes, hipStream_t s) {
  if (items <= 0) return hipSuccess;
  hipLaunchKernelGGL(jacobi_single_kernel, dim3(items), dim3(512), lds_bytes, s, items_dev,
                     max_sweeps, eps_scale);
  return hipGetLastError();
}

// sigma_i = ||a_i||, stable descending sort, k = min(cap, #{sigma > cutoff ||sigma||}) >= 1,
// normalised output vectors (Algorithm 1's final loop and sort; truncation of Eq. svd).
// FIN_GATE: no vector (zero) for a sigma that is round-off.  Algorithm 1 leaves
// pairs below eps^2 ||A||_F^2 as they are, so the vectors of sigma_i and sigma_1
// overlap by up to that over sigma_1 sigma_i: 1e-12 at 2^-53 ||sigma||, but any
// angle further down, where a normalised vector would count sigma_1's direction
// once more.
__global__ __launch_bounds__(1024) void finalize_kernel(const FinItem* items) {
  __shared__ double sig[1024];
  __shared__ int perm[1024];
  __shared__ int s_k;
  __shared__ double s_inv, s_least;
  const FinItem it = items[blockIdx.x];
  const int n = it.n, m = it.m;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int v = wave; v < n; v += 16) {
    double acc = 0.0;
    for (int e = lane; e < m; e += 64) {
      const double2 x = it.w[(size_t)v * m + e];
      acc += x.x * x.x + x.y * x.y;
    }
    acc = wave_sum(acc);
    if (lane == 0) sig[v] = sqrt(acc);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += blockDim.x) perm[i] = i;  // (a NaN leaves ranks unset)
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const double si = sig[i];
    int r = 0;
    for (int j = 0; j < n; ++j) {
      const double sj = sig[j];
      r += (sj > si) || (sj == si && j < i);
    }
    perm[r] = i;
  }
  __syncthreads();
  // sums over the values: one wave, lane l takes l, l + 64, ...
  if (threadIdx.x < 64) {
    double tot = 0.0;
    for (int a = lane; a < n; a += 64) tot += sig[a] * sig[a];
    tot = wave_sum(tot);
    const double nrm = sqrt(tot);
    int k = 0;
    for (int a = lane; a < n; a += 64) k += sig[a] > it.cutoff * nrm ? 1 : 0;
    k = (int)wave_sum((double)k);
    k = min(max(k, 1), it.cap);
    double kept2 = 0.0, disc2 = 0.0;
    for (int a = lane; a < n; a += 64) {
      const double sv = sig[perm[a]];
      if (a < k) kept2 += sv * sv;
      else disc2 += sv * sv;
    }
    kept2 = wave_sum(kept2);
    disc2 = wave_sum(disc2);
    const double kept = sqrt(kept2);
    const bool bad = !isfinite(tot) || !(kept > 0.0) || !isfinite(kept);
    if (lane == 0) {
      *it.status_out = bad ? 1 : 0;
      s_inv = bad ? 0.0 : 1.0 / kept;
      *it.k_out = k;
      *it.scale_out = s_inv;
      *it.disc_out = tot > 0.0 ? disc2 / tot : 0.0;
      s_k = k;
      s_least = it.mode == FIN_GATE ? 0x1p-53 * nrm : 0.0;
    }
  }
  __syncthreads();
  const int k = s_k;
  const double inv = s_inv;
  if (it.mode == FIN_LEFT) {
    for (int idx = threadIdx.x; idx < m * k; idx += blockDim.x) {
      const int e = idx / k, a = idx - (idx / k) * k;
      const double sv = sig[perm[a]];
      const double2 x = it.w[(size_t)perm[a] * m + e];
      it.vec_out[idx] = sv > 0.0 ? make_double2(x.x / sv, x.y / sv) : make_double2(0.0, 0.0);
    }
  } else {
    for (int a = threadIdx.x; a < k; a += blockDim.x) it.lam_out[a] = sig[perm[a]] * inv;
    const int half = m / 2;
    for (int idx = threadIdx.x; idx < k * m; idx += blockDim.x) {
      const int a = idx / m, e = idx - (idx / m) * m;
      const int s = e / half, r = e - s * half;
      const double sv = sig[perm[a]];
      const double2 x = it.w[(size_t)perm[a] * m + e];
      it.vec_out[((size_t)s * k + a) * half + r] =
          sv > s_least ? make_double2(x.x / sv, x.y / sv) : make_double2(0.0, 0.0);
    }
  }
}

hipError_t launch_finalize(const FinItem* items_dev, int items, hipStream_t s) {
  if (items <= 0) return hipSuccess;
  hipLaunchKernelGGL(finalize_kernel, dim3(items), dim3(1024), 0, s, items_dev);
  return hipGetLastError();
}

// =================================================================== Eq. (Bl)

struct TruncP {
  using T = double;
  using Ctx = TruncItem;
  static constexpr bool A_CONTIG_K = true, B_CONTIG_N = false, REAL_ONLY = false;
  const TruncItem* items;
  __device__ Ctx context(int i) const {
    TruncItem t = items[i];
    if (t.k_dev) t.k = min(t.k, *t.k_dev);
    return t;
  }
  __device__ static void dims(const Ctx& c, int& M, int& N, int& K) {
    M = c.rows;
    N = c.k;
    K = 2 * c.dr;
  }
  using RowA = const double2*;
  using ColB = const double2*;
  __device__ static RowA rowA(const Ctx& c, int i) { return c.c + (size_t)i * (2 * c.dr); }
  __device__ static ColB colB(const Ctx& c, int j) { return c.v + (size_t)j * c.dr; }
  __device__ static double2 loadA(const Ctx&, RowA r, int, int k) { return r[k]; }
  __device__ static double2 loadB(const Ctx& c, ColB b, int k, int) {
    const int s = k >= c.dr;
    const double2 v = b[(size_t)s * c.k * c.dr + (k - s * c.dr)];
    return make_double2(v.x, -v.y);
  }
  __device__ static void store(const Ctx& c, int i, int j, double re, double im) {
    const double sc = *c.scale;
    c.out[(size_t)i * c.k + j] = make_double2(re * sc, im * sc);
  }
};

hipError_t launch_trunc(const TruncItem* items_dev, int items, int max_rows, int max_k,
                        hipStream_t s) {
  TruncP p{items_dev};
  return launch_cgemm<64, 64, 16>(p, items, max_rows, max_k, s);
}

// =================================================================== canonical form

struct CanonLeftP {  // W[beta][(s,alpha)] = sum_g B[s][g][beta] T[alpha][g]
  using T = double;
  using Ctx = CanonLeftItem;
  static constexpr bool A_CONTIG_K = false, B_CONTIG_N = false, REAL_ONLY = false;
  const CanonLeftItem* items;
  __device__ Ctx context(int i) const { return items[i]; }
  __device__ static void dims(const Ctx& c, int& M, int& N, int& K) {
    M = c.db;
    N = c.r;
    K = c.dg;
  }
  using RowA = const double2*;
  using ColB = const double2*;
  __device__ static RowA rowA(const Ctx& c, int i) { return c.b + (size_t)c.s * c.dg * c.db + i; }
  __device__ static ColB colB(const Ctx& c, int j) { return c.t + (size_t)j * c.dg; }
  __device__ static double2 loadA(const Ctx& c, RowA r, int, int k) { return r[(size_t)k * c.db]; }
  __device__ static double2 loadB(const Ctx&, ColB b, int k, int) { return b[k]; }
  __device__ static void store(const Ctx& c, int i, int j, double re, double im) {
    c.w[(size_t)i * (2 * c.r) + c.s * c.r + j] = make_double2(re, im);
  }
};

struct CanonCarryLeftP {  // T'[a][beta] = sum_e conj(A[e][a]) W0[beta][e]
  using T = double;
  using Ctx = CanonCarryLeftItem;
  static constexpr bool A_CONTIG_K = false, B_CONTIG_N = false, REAL_ONLY = false;
  const CanonCarryLeftItem* items;
  __device__ Ctx context(int i) const { return items[i]; }
  __device__ static void dims(const Ctx& c, int& M, int& N, int& K) {
    M = c.k;
    N = c.db;
    K = c.m;
  }
  using RowA = const double2*;
  using ColB = const double2*;
  __device__ static RowA rowA(const Ctx& c, int i) { return c.a + i; }
  __device__ static ColB colB(const Ctx& c, int j) { return c.w0 + (size_t)j * c.m; }
  __device__ static double2 loadA(const Ctx& c, RowA r, int, int k) {
    const double2 v = r[(size_t)k * c.k];
    return make_double2(v.x, -v.y);
  }
  __device__ static double2 loadB(const Ctx&, ColB b, int k, int) { return b[k]; }
  __device__ static void store(const Ctx& c, int i, int j, double re, double im) {
    c.t[(size_t)i * c.db + j] = make_double2(re, im);
  }
};

struct CanonRightP {  // W[alpha][(s,b')] = sum_beta A[s][alpha][beta] T[beta][b']
  using T = double;
  using Ctx = CanonRightItem;
  static constexpr bool A_CONTIG_K = true, B_CONTIG_N = true, REAL_ONLY = false;
  const CanonRightItem* items;
  __device__ Ctx context(int i) const { return items[i]; }
  __device__ static void dims(const Ctx& c, int& M, int& N, int& K) {
    M = c.dl;
    N = c.r;
    K = c.dm;
  }
  using RowA = const double2*;
  using ColB = const double2*;
  __device__ static RowA rowA(const Ctx& c, int i) { return c.a + ((size_t)c.s * c.dl + i) * c.dm; }
  __device__ static ColB colB(const Ctx& c, int j) { return c.t + j; }
  __device__ static double2 loadA(const Ctx&, RowA r, int, int k) { return r[k]; }
  __device__ static double2 loadB(const Ctx& c, ColB b, int k, int) { return b[(size_t)k * c.r]; }
  __device__ static void store(const Ctx& c, int i, int j, double re, double im) {
    c.w[(size_t)i * (2 * c.r) + c.s * c.r + j] = make_double2(re, im);
  }
};

hipError_t launch_canon_left(const CanonLeftItem* items_dev, int items, int max_db, int max_r,
                             hipStream_t s) {
  CanonLeftP p{items_dev};
  return launch_cgemm<64, 64, 16>(p, items, max_db, max_r, s);
}
hipError_t launch_canon_carry_left(const CanonCarryLeftItem* items_dev, int items, int max_k,
                                   int max_db, hipStream_t s) {
  CanonCarryLeftP p{items_dev};
  return launch_cgemm<64, 64, 16>(p, items, max_k, max_db, s);
}
hipError_t launch_canon_right(const CanonRightItem* items_dev, int items, int max_dl, int max_r,
                              hipStream_t s) {
  CanonRightP p{items_dev};
  return launch_cgemm<64, 64, 16>(p, items, max_dl, max_r, s);
}

__global__ __launch_bounds__(256) void fro2_kernel(const double2* w, int count, double* out) {
  double acc = 0.0;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < count; i += gridDim.x * 256) {
    const double2 x = w[i];
    acc += x.x * x.x + x.y * x.y;
  }
  acc = wave_sum(acc);
  __shared__ double part[4];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) atomicAdd(out, part[0] + part[1] + part[2] + part[3]);
}

hipError_t launch_fro2(const double2* w, int count, double* out, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  int blocks = cdiv(count, 256);
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(fro2_kernel, dim3(blocks), dim3(256), 0, s, w, count, out);
  return hipGetLastError();
}

__global__ void copy_kernel(double2* dst, const double2* src, size_t count) {
  for (size_t i = blockIdx.x * (size_t)256 + threadIdx.x; i < count; i += (size_t)gridDim.x * 256)
    dst[i] = src[i];
}

hipError_t launch_copy(double2* dst, const double2* src, size_t count, hipStream_t s) {
  if (count == 0) return hipSuccess;
  size_t blocks = (count + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(copy_kernel, dim3((unsigned)blocks), dim3(256), 0, s, dst, src, count);
  return hipGetLastError();
}

// Several device-to-device copies in one launch: block row y takes item y,
// 2048 doubles per block along x.
__global__ __launch_bounds__(256) void copy_list_kernel(const RawCopy* items) {
  const RawCopy it = items[blockIdx.y];
  const long long base = (long long)blockIdx.x * 2048;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const long long i = base + 2 * (u * 256 + (int)threadIdx.x);
    if (i + 1 < it.words) *(double2*)(it.dst + i) = *(const double2*)(it.src + i);
    else if (i < it.words) it.dst[i] = it.src[i];
  }
}

hipError_t launch_copy_list(const RawCopy* items, int count, long long max_words, hipStream_t s) {
  if (count <= 0 || max_words <= 0) return hipSuccess;
  if (count > 65535) return hipErrorInvalidValue;
  hipLaunchKernelGGL(copy_list_kernel, dim3(cdiv(max_words, 2048), count), dim3(256), 0, s, items);
  return hipGetLastError();
}

// =================================================================== fixed scratch

// Device scratch of the entry point that allocates nothing
// (mps_jacobi_svd_noalloc).  Each device holds its own copy of the array at
// its own address; host code reaches it only through the address
// hipGetSymbolAddress returns for the current device, looked up once per
// device and kept.  Every call on a device shares its copy.
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {
constexpr int kScratchDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kScratchDevices] = {};
}  // namespace

hipError_t scratch_address(void** out) {
  *out = nullptr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kScratchDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

// Zero-fill of a device region (a kernel, not a memset node: callers may
// capture it in a graph).
__global__ void zero_kernel(uint64_t* dst, size_t words) {
  for (size_t i = blockIdx.x * (size_t)256 + threadIdx.x; i < words; i += (size_t)gridDim.x * 256)
    dst[i] = 0;
}

hipError_t launch_zero(void* dst, size_t bytes, hipStream_t s) {
  const size_t words = (bytes + 7) / 8;
  if (words == 0) return hipSuccess;
  size_t blocks = (words + 255) / 256;
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(zero_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (uint64_t*)dst, words);
  return hipGetLastError();
}

// One site of the statevector contraction of Eq. (mps):
//   out[(a, s)][beta] = sum_alpha in[a][alpha] B^s[alpha][beta],
// `in` holding `amps` rows of D_l amplitudes-with-open-bond, `out` 2 amps rows
// of D_r.  Row index a is the bit string of the sites already contracted,
// the earliest site most significant, so qubit 0 ends as the top bit.
__global__ void sv_site_kernel(const double2* in, const double2* b, double2* out, int64_t amps, int dl,
                               int dr) {
  const int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x;
  const int64_t total = amps * 2 * dr;
  if (i >= total) return;
  const int beta = (int)(i % dr);
  const int64_t as = i / dr;
  const int sbit = (int)(as & 1);
  const int64_t a = as >> 1;
  const double2* row = in + a * dl;
  const double2* col = b + (size_t)sbit * dl * dr + beta;
  double re = 0.0, im = 0.0;
  for (int al = 0; al < dl; ++al) {
    const double2 x = row[al], y = col[(size_t)al * dr];
    re += x.x * y.x - x.y * y.y;
    im += x.x * y.y + x.y * y.x;
  }
  out[i] = make_double2(re, im);
}

hipError_t launch_sv_site(const double2* in, const double2* b, double2* out, int64_t amps, int dl, int dr,
                          hipStream_t s) {
  const int64_t total = amps * 2 * dr;
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(sv_site_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, in, b, out, amps,
                     dl, dr);
  return hipGetLastError();
}

__global__ void fill_ident_kernel(double2* dst, int d) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < d * d) dst[i] = make_double2((i / d) == (i % d) ? 1.0 : 0.0, 0.0);
}

hipError_t launch_fill_ident(double2* dst, int d, hipStream_t s) {
  if (d <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_ident_kernel, dim3(cdiv((long long)d * d, 256)), dim3(256), 0, s, dst, d);
  return hipGetLastError();
}

// =================================================================== Eq. (expec2)

// The segment that holds item i, by all lanes of a wave together: every step
// tests 64 ends at once (one load for up to 64 segments; END: par_end or
// chi_end).  first: the segment's first item.
template <int EnvSeg::*END>
__device__ __forceinline__ int find_segment(const EnvSeg* segs, int n, int i, int& first) {
  const int lane = threadIdx.x & 63;
  int lo = 0, len = n;
  while (len > 1) {
    const int step = (len + 63) / 64, p = lo + (lane + 1) * step - 1;
    const bool before = p < lo + len && segs[p].*END <= i;
    const int skip = __popcll(__ballot(before)) * step;
    lo += skip;
    len = min(step, len - skip);
  }
  lo = __builtin_amdgcn_readfirstlane(lo);
  first = lo ? segs[lo - 1].*END : 0;
  return lo;
}

// X = L [A^0 | A^1]: (Dl x Dl)(Dl x 2Dr); one item per parent, the site A and
// the dims the launch's or (merged launches) the segment's.
template <typename TT>
struct EnvG1P {
  using T = TT;
  using C2 = typename cplx_of<TT>::type;
  struct Ctx {
    const C2* l;
    C2* x;
    const C2* site;
    int dl, dr;
  };
  static constexpr bool A_CONTIG_K = true, B_CONTIG_N = true, REAL_ONLY = false;
  const EnvParent<C2>* items;
  const C2* site;
  int dl, dr;
  const EnvSeg* segs = nullptr;
  int n_segs = 0;
  __device__ Ctx context(int i) const {
    if (segs) {
      int base;
      const int s = find_segment<&EnvSeg::par_end>(segs, n_segs, i, base);
      const EnvParent<C2> e = ((const EnvParent<C2>*)segs[s].par)[i - base];
      return Ctx{e.l, e.x, (const C2*)segs[s].site, segs[s].dl, segs[s].dr};
    }
    const EnvParent<C2> e = items[i];
    return Ctx{e.l, e.x, site, dl, dr};
  }
  __device__ static void dims(const Ctx& c, int& M, int& N, int& K) {
    M = c.dl;
    N = 2 * c.dr;
    K = c.dl;
  }
  using RowA = const C2*;
  using ColB = const C2*;
  __device__ static RowA rowA(const Ctx& c, int i) { return c.l + (size_t)i * c.dl; }
  __device__ static ColB colB(const Ctx& c, int j) {
    const int s = j >= c.dr;
    return c.site + (size_t)s * c.dl * c.dr + (j - s * c.dr);
  }
  __device__ static C2 loadA(const Ctx&, RowA r, int, int k) { return r[k]; }
  __device__ static C2 loadB(const Ctx& c, ColB b, int k, int) { return b[(size_t)k * c.dr]; }
  // Eight consecutive k (k + 7 < K) for the 16-bit split GEMM; the return
  // value is the operation on the split planes that turns the loaded values
  // into the operand (SPLIT_SWAP, SPLIT_NEG_RE, SPLIT_NEG_IM bits; none here).
  __device__ __forceinline__ static int loadA8(const Ctx&, RowA r, int, int k, C2 (&o)[8]) {
#pragma unroll
    for (int t = 0; t < 8; ++t) o[t] = r[k + t];
    return 0;
  }
  __device__ __forceinline__ static int loadB8(const Ctx& c, ColB b, int k, int, C2 (&o)[8]) {
    const C2* q = b + (size_t)k * c.dr;
#pragma unroll
    for (int t = 0; t < 8; ++t) o[t] = q[(size_t)t * c.dr];
    return 0;
  }
  __device__ static void store(const Ctx& c, int i, int j, TT re, TT im) {
    C2 v;
    v.x = re;
    v.y = im;
    c.x[(size_t)i * (2 * c.dr) + j] = v;
  }
};

// L' = sum_s A^{s+} Y^s with Y^s = sum_s' sigma_{ss'} X^{s'}: a block swap
// (X, Y letters) and a phase (Y: -i, +i; Z: +1, -1) folded into the B fetch.
template <typename TT>
struct EnvG2P {
  using T = TT;
  using C2 = typename cplx_of<TT>::type;
  struct Ctx {
    const C2* x;
    C2* out;
    const C2* site;
    int dl, dr, letter;
  };
  static constexpr bool A_CONTIG_K = false, B_CONTIG_N = true, REAL_ONLY = false;
  const EnvChild<C2>* items;
  const C2* site;
  int dl, dr;
  const EnvSeg* segs = nullptr;
  int n_segs = 0;
  __device__ Ctx context(int i) const {
    if (segs) {
      int base;
      const int s = find_segment<&EnvSeg::chi_end>(segs, n_segs, i, base);
      const EnvChild<C2> e = ((const EnvChild<C2>*)segs[s].chi)[i - base];
      return Ctx{e.x, e.out, (const C2*)segs[s].site, segs[s].dl, segs[s].dr, e.letter};
    }
    const EnvChild<C2> e = items[i];
    return Ctx{e.x, e.out, site, dl, dr, e.letter};
  }
  __device__ static void dims(const Ctx& c, int& M, int& N, int& K) {
    M = c.dr;
    N = c.dr;
    K = 2 * c.dl;
  }
  using RowA = const C2*;
  using ColB = const C2*;
  __device__ static RowA rowA(const Ctx& c, int i) { return c.site + i; }
  __device__ static ColB colB(const Ctx& c, int j) { return c.x + j; }
  __device__ static C2 loadA(const Ctx& c, RowA r, int, int k) {
    // element (beta, (s, alpha)) of [A^0+ | A^1+] is conj(A[s][alpha][beta]); k = s*dl + alpha
    C2 v = r[(size_t)k * c.dr];
    v.y = -v.y;
    return v;
  }
  __device__ static C2 loadB(const Ctx& c, ColB b, int k, int) {
    const int s = k >= c.dl;
    const int a = k - s * c.dl;
    const int flip = (c.letter == 1 || c.letter == 2) ? 1 : 0;
    const C2 v = b[(size_t)a * (2 * c.dr) + (s ^ flip) * c.dr];
    C2 o = v;
    if (c.letter == 2) {  // Y: s=0 -> -i X^1, s=1 -> +i X^0
      if (s == 0) { o.x = v.y; o.y = -v.x; }
      else { o.x = -v.y; o.y = v.x; }
    } else if (c.letter == 3 && s == 1) {
      o.x = -v.x;
      o.y = -v.y;
    }
    return o;
  }
  // Eight consecutive k as in EnvG1P: the conjugation, and the letter's
  // phase when all eight share one s, become sign flips and a swap of the
  // split planes (exact: the split commutes with negation); eight k across
  // the s boundary are loaded one by one.
  __device__ __forceinline__ static int loadA8(const Ctx& c, RowA r, int, int k, C2 (&o)[8]) {
    const C2* q = r + (size_t)k * c.dr;
#pragma unroll
    for (int t = 0; t < 8; ++t) o[t] = q[(size_t)t * c.dr];
    return SPLIT_NEG_IM;
  }
  __device__ __forceinline__ static int loadB8(const Ctx& c, ColB b, int k, int j, C2 (&o)[8]) {
    const int s = k >= c.dl;
    const int a = k - s * c.dl;
    if (a + 7 >= c.dl) {
#pragma unroll
      for (int t = 0; t < 8; ++t) o[t] = loadB(c, b, k + t, j);
      return 0;
    }
    const int flip = (c.letter == 1 || c.letter == 2) ? 1 : 0;
    const C2* q = b + (size_t)a * (2 * c.dr) + (s ^ flip) * c.dr;
#pragma unroll
    for (int t = 0; t < 8; ++t) o[t] = q[(size_t)t * (2 * c.dr)];
    if (c.letter == 2) return s == 0 ? (SPLIT_SWAP | SPLIT_NEG_IM) : (SPLIT_SWAP | SPLIT_NEG_RE);
    if (c.letter == 3 && s == 1) return SPLIT_NEG_RE | SPLIT_NEG_IM;
    return 0;
  }
  __device__ static void store(const Ctx& c, int i, int j, TT re, TT im) {
    C2 v;
    v.x = re;
    v.y = im;
    c.out[(size_t)i * c.dr + j] = v;
  }
};

// The address of a wave's operand as a scalar; load_g reads from memory at it.
__device__ __forceinline__ size_t uniform_addr(const void* p) {
  const size_t v = (size_t)p;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v), hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
  return (size_t)hi << 32 | lo;
}
template <typename T>
__device__ __forceinline__ typename cplx_of<T>::type load_g(size_t base, size_t off) {
  typedef T vec __attribute__((ext_vector_type(2)));
  const vec v = *(const __attribute__((address_space(1))) vec*)((const __attribute__((address_space(1))) char*)base + off);
  typename cplx_of<T>::type o;
  o.x = v.x;
  o.y = v.y;
  return o;
}
__device__ __forceinline__ double flip_sign(double v, unsigned mask) {
  return __hiloint2double(__double2hiint(v) ^ (int)mask, __double2loint(v));
}
__device__ __forceinline__ float flip_sign(float v, unsigned mask) { return __uint_as_float(__float_as_uint(v) ^ mask); }

// The environment GEMMs (c128, c64): bound by the matrix cores once the loop
// has little else in it.  cgemm_kernel's loads carry the letter's phase, the s
// boundary and the edges as branches per element, and a branch around a load
// makes the loop wait for it; here a wave loads whole rows of both operands, so
// the row's s, phase and sign are scalars, rows past the edge are clamped
// (their products are never stored) and only a last partial chunk is masked.
// Two LDS buffers and one barrier per chunk, complex elements interleaved (one
// read per fragment).  Same products in the same order as cgemm_kernel.  50
// qubits D = 256 c128: 225 -> 205 ms (57 -> 64 TFLOP/s of the 73 a large FP64
// matrix product reaches); 28 qubits D = 512 c64: 74 -> 63 ms of updates (105
// -> 124 TFLOP/s of 151).
template <class P, int HALF, int BM, int BN, int BK>
__global__ __launch_bounds__(256, 2) void env_gemm_kernel(P p, int tiles_m, int tiles_n, int total, int g8) {
  using T = typename P::T;
  using C2 = typename cplx_of<T>::type;
  using Acc = typename acc_of<T>::type;
  constexpr int RA = BM / 64, RB = BN / 64, EK = BK / 4;  // loads per row, rows per wave and chunk
  constexpr int FM = BM / 32, FN = BN / 32;
  __shared__ C2 As[2][BK][BM + 1];
  __shared__ C2 Bs[2][BK][BN + 1];

  const int logical = xcd_remap(blockIdx.x, g8);
  if (logical >= total) return;
  const int per_item = tiles_m * tiles_n;
  const int item = logical / per_item;
  const int t = logical - item * per_item;
  const int tm = t / tiles_n;
  const int m0 = tm * BM, n0 = (t - tm * tiles_n) * BN;
  const typename P::Ctx ctx = p.context(item);
  const int dl = __builtin_amdgcn_readfirstlane(ctx.dl), dr = __builtin_amdgcn_readfirstlane(ctx.dr);
  constexpr size_t EL = sizeof(C2);
  const size_t site = uniform_addr(ctx.site);
  size_t env;  // HALF 1: L, HALF 2: X
  int M, N, K, letter = 0;
  C2* out;
  if constexpr (HALF == 1) {
    env = uniform_addr(ctx.l);
    out = ctx.x;
    M = K = dl;
    N = 2 * dr;
  } else {
    env = uniform_addr(ctx.x);
    letter = __builtin_amdgcn_readfirstlane(ctx.letter);
    out = ctx.out;
    M = N = dr;
    K = 2 * dl;
  }
  if (m0 >= M || n0 >= N) return;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave >> 1) * (BM / 2), wn = (wave & 1) * (BN / 2);
  const int lr = lane & 15, lk = lane >> 4;
  const int flip = (letter == 1 || letter == 2) ? 1 : 0;
  const bool swap = letter == 2;

  // Per-lane offsets in bytes.  HALF 1 loads A with k along the lanes (k is
  // contiguous in memory: k = tid % BK, rows tid / BK + ...); every other load
  // takes a row of 64 at k = wave + 4 e.
  constexpr int AK = 256 / BK;
  const int ak = tid % BK, ai = tid / BK;
  unsigned oa[HALF == 1 ? EK * RA : RA];
  if constexpr (HALF == 1) {
#pragma unroll
    for (int e = 0; e < EK * RA; ++e)
      oa[e] = ((unsigned)min(ai + e * AK, M - 1 - m0) * dl + ak) * (unsigned)EL;
    env += (size_t)m0 * dl * EL;
  } else {
#pragma unroll
    for (int h = 0; h < RA; ++h) oa[h] = (unsigned)min(m0 + lane + 64 * h, M - 1) * (unsigned)EL;
  }
  size_t ob[RB];
#pragma unroll
  for (int h = 0; h < RB; ++h) {
    const int j = min(n0 + lane + 64 * h, N - 1), s = HALF == 1 && j >= dr;
    ob[h] = HALF == 1 ? (s ? (size_t)dl * dr + (j - dr) : (size_t)j) * EL : (unsigned)j * (unsigned)EL;
  }

  // Loads and LDS stores of the chunk at k0; loads past K take the last k,
  // which put() replaces by zeros (MASK: the chunk reaches past K).
  C2 ra[EK * RA], rb[EK * RB];
  auto load = [&](int k0) {
    if constexpr (HALF == 1) {
      const unsigned back = (unsigned)max(k0 + ak - (K - 1), 0) * (unsigned)EL;
#pragma unroll
      for (int e = 0; e < EK * RA; ++e) ra[e] = load_g<T>(env, (size_t)k0 * EL + oa[e] - back);
    }
#pragma unroll
    for (int e = 0; e < EK; ++e) {
      const int k = min(k0 + wave + 4 * e, K - 1);
      const size_t srow = site + (size_t)k * dr * EL;
      if constexpr (HALF == 1) {
#pragma unroll
        for (int h = 0; h < RB; ++h) rb[e * RB + h] = load_g<T>(srow, ob[h]);
      } else {
        const int s = k >= dl ? 1 : 0, row = 2 * (k - s * dl) + (flip ? 1 - s : s);
        const size_t xrow = env + (size_t)row * dr * EL;
#pragma unroll
        for (int h = 0; h < RA; ++h) ra[e * RA + h] = load_g<T>(srow, oa[h]);
#pragma unroll
        for (int h = 0; h < RB; ++h) rb[e * RB + h] = load_g<T>(xrow, ob[h]);
      }
    }
  };
  auto put = [&](int b, int k0, auto mask) {
    constexpr bool MASK = decltype(mask)::value;
    auto keep = [](C2 v, bool in) {
      if (MASK) {
        v.x = in ? v.x : T(0);
        v.y = in ? v.y : T(0);
      }
      return v;
    };
    if constexpr (HALF == 1) {
#pragma unroll
      for (int e = 0; e < EK * RA; ++e) As[b][ak][ai + e * AK] = keep(ra[e], k0 + ak < K);
    }
#pragma unroll
    for (int e = 0; e < EK; ++e) {
      const int kk = wave + 4 * e;
      const bool in = k0 + kk < K, s1 = k0 + kk >= dl;
      if constexpr (HALF == 2) {
#pragma unroll
        for (int h = 0; h < RA; ++h) {
          C2 v = keep(ra[e * RA + h], in);
          v.y = -v.y;
          As[b][kk][lane + 64 * h] = v;
        }
      }
      // Y: s=0 -> -i X^1, s=1 -> +i X^0;  Z: s=1 -> -X^1
      const unsigned nx = s1 && letter >= 2 ? 0x80000000u : 0u;
      const unsigned ny = (letter == 2 && !s1) || (letter == 3 && s1) ? 0x80000000u : 0u;
#pragma unroll
      for (int h = 0; h < RB; ++h) {
        C2 v = keep(rb[e * RB + h], in);
        if constexpr (HALF == 2) {
          const T re = swap ? v.y : v.x, im = swap ? v.x : v.y;
          v.x = flip_sign(re, nx);
          v.y = flip_sign(im, ny);
        }
        Bs[b][kk][lane + 64 * h] = v;
      }
    }
  };
  auto stage = [&](int b, int k0) {
    if (k0 + BK <= K) put(b, k0, std::false_type{});
    else put(b, k0, std::true_type{});
  };

  Acc acc_r[FM][FN], acc_i[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc_r[i][j][v] = acc_i[i][j][v] = T(0);

  load(0);
  stage(0, 0);
  load(BK);
  lds_barrier();
  int b = 0;
  for (int k0 = 0; k0 < K; k0 += BK, b ^= 1) {
    if (k0 + BK < K) stage(b ^ 1, k0 + BK);  // its readers passed the last barrier
    load(k0 + 2 * BK);  // unconditional (past K: clamped): a branch here makes the loop wait for it
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      C2 a[FM], c[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i) a[i] = As[b][kk + lk][wm + i * 16 + lr];
#pragma unroll
      for (int j = 0; j < FN; ++j) c[j] = Bs[b][kk + lk][wn + j * 16 + lr];
      // the two products of one accumulator are kept apart: the second waits for the first
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          acc_r[i][j] = mfma_16x16x4(a[i].x, c[j].x, acc_r[i][j]);
          acc_i[i][j] = mfma_16x16x4(a[i].x, c[j].y, acc_i[i][j]);
        }
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          acc_r[i][j] = mfma_16x16x4(-a[i].y, c[j].y, acc_r[i][j]);
          acc_i[i][j] = mfma_16x16x4(a[i].y, c[j].x, acc_i[i][j]);
        }
    }
    lds_barrier();
  }

#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = m0 + wm + i * 16 + acc_row<T>(lk, v);
        const int col = n0 + wn + j * 16 + lr;
        if (row < M && col < N) {
          C2 o;
          o.x = acc_r[i][j][v];
          o.y = acc_i[i][j][v];
          out[(size_t)row * N + col] = o;
        }
      }
}

template <int BM, int BN, int BK, class P>
hipError_t launch_env_gemm(const P& p, int count, int m, int n, hipStream_t s) {
  if (count <= 0 || m <= 0 || n <= 0) return hipSuccess;
  constexpr int HALF = P::A_CONTIG_K ? 1 : 2;
  const int tm = cdiv(m, BM), tn = cdiv(n, BN);
  const long long total = (long long)count * tm * tn;
  if (total > 0x7fffff00LL) return hipErrorInvalidValue;
  const int g8 = (int)((total + 7) / 8 * 8);
  hipLaunchKernelGGL((env_gemm_kernel<P, HALF, BM, BN, BK>), dim3(g8), dim3(256), 0, s, p, tm, tn, (int)total, g8);
  return hipGetLastError();
}

// FP64: 64 x 64 x 8, four workgroups per compute unit (50 qubits D = 256:
// 205 ms; 64 x 64 x 16 with two 212, 128 x 64 x 8 with two 208).  FP32: 128 x 64
// where that pads no further rows and still gives four workgroups per compute
// unit (28 qubits D = 512: 63 ms of updates per call, 66 in 64 x 64 tiles).
template <class P>
hipError_t launch_env_64(const P& p, int count, int m, int n, hipStream_t s) {
  if constexpr (sizeof(typename P::T) == 8) return launch_env_gemm<64, 64, 8>(p, count, m, n, s);
  else if (cdiv(m, 64) % 2 == 0 && (long long)count * cdiv(m, 128) * cdiv(n, 64) >= 1024)
    return launch_env_gemm<128, 64, 8>(p, count, m, n, s);
  else return launch_env_gemm<64, 64, 16>(p, count, m, n, s);
}

// One environment GEMM with tile kEnvTileShape[tile] (all give bitwise-identical
// results: every output element accumulates its K range in the same order of
// 16x16x4 steps whatever the tile).
template <class P>
hipError_t launch_env_tile(const P& p, int tile, int count, int m, int n, hipStream_t s) {
  switch (tile) {
    case 0: return launch_env_64(p, count, m, n, s);
    case 1: return launch_cgemm<32, 32, 16>(p, count, m, n, s);
    case 2: return launch_cgemm<128, 64, 16>(p, count, m, n, s);
    case 3: return launch_cgemm<64, 128, 16>(p, count, m, n, s);
    case 4: return launch_cgemm<64, 64, 32>(p, count, m, n, s);
    case 5: return launch_cgemm<32, 64, 16>(p, count, m, n, s);
    case 6: return launch_cgemm<128, 128, 16>(p, count, m, n, s);
    case 7: return launch_cgemm<128, 128, 8>(p, count, m, n, s);
    default: return hipErrorInvalidValue;
  }
}
static_assert(kEnvTiles == 8, "launch_env_tile covers every tile shape");

hipError_t launch_env_gemm1_c128(const EnvParent<double2>* items, int count, const double2* site,
                                 int dl, int dr, hipStream_t s, int tile) {
  EnvG1P<double> p{items, site, dl, dr};
  return launch_env_tile(p, tile, count, dl, 2 * dr, s);
}
hipError_t launch_env_gemm2_c128(const EnvChild<double2>* items, int count, const double2* site,
                                 int dl, int dr, hipStream_t s, int tile) {
  EnvG2P<double> p{items, site, dl, dr};
  return launch_env_tile(p, tile, count, dr, dr, s);
}
hipError_t launch_env_gemm1_c64(const EnvParent<float2>* items, int count, const float2* site,
                                int dl, int dr, hipStream_t s, int tile) {
  EnvG1P<float> p{items, site, dl, dr};
  return launch_env_tile(p, tile, count, dl, 2 * dr, s);
}
hipError_t launch_env_gemm2_c64(const EnvChild<float2>* items, int count, const float2* site,
                                int dl, int dr, hipStream_t s, int tile) {
  EnvG2P<float> p{items, site, dl, dr};
  return launch_env_tile(p, tile, count, dr, dr, s);
}

// split precisions: FP32 environments, 16-bit matrix cores, FP32 accumulation
hipError_t launch_env_gemm1_split(const EnvParent<float2>* items, int count, const float2* site, int dl,
                                  int dr, int f16, hipStream_t s) {
  EnvG1P<float> p{items, site, dl, dr};
  return f16 ? launch_cgemm_split<_Float16, 64, 64>(p, count, dl, 2 * dr, s)
             : launch_cgemm_split<__bf16, 64, 64>(p, count, dl, 2 * dr, s);
}
hipError_t launch_env_gemm2_split(const EnvChild<float2>* items, int count, const float2* site, int dl,
                                  int dr, int f16, hipStream_t s) {
  EnvG2P<float> p{items, site, dl, dr};
  return f16 ? launch_cgemm_split<_Float16, 64, 64>(p, count, dr, dr, s)
             : launch_cgemm_split<__bf16, 64, 64>(p, count, dr, dr, s);
}

// Merged launches: c128 and c64 take the 32 x 32 tile where 64 x 64 ones would
// leave the chip idle (two per compute unit; at D = 64 and 50 items the two
// halves take 11 + 21 us in 64 x 64 tiles).
// A single segment goes by value: looking it up in memory first delays every
// workgroup by two dependent loads (50 qubits D = 256 split-F16 3% slower).
template <typename T>
EnvG1P<T> env_p1(const EnvMerged& m) {
  using C2 = typename cplx_of<T>::type;
  if (m.n_segs > 1) return EnvG1P<T>{nullptr, nullptr, 0, 0, m.segs, m.n_segs};
  return EnvG1P<T>{(const EnvParent<C2>*)m.one.par, (const C2*)m.one.site, m.one.dl, m.one.dr};
}
template <typename T>
EnvG2P<T> env_p2(const EnvMerged& m) {
  using C2 = typename cplx_of<T>::type;
  if (m.n_segs > 1) return EnvG2P<T>{nullptr, nullptr, 0, 0, m.segs, m.n_segs};
  return EnvG2P<T>{(const EnvChild<C2>*)m.one.chi, (const C2*)m.one.site, m.one.dl, m.one.dr};
}

template <typename T>
hipError_t env_merged_t(const EnvMerged& m, hipStream_t s) {
  const EnvG1P<T> p1 = env_p1<T>(m);
  const EnvG2P<T> p2 = env_p2<T>(m);
  const long long t1 = (long long)m.n_par * cdiv(m.max_dl, 64) * cdiv(2 * m.max_dr, 64);
  const long long t2 = (long long)m.n_chi * cdiv(m.max_dr, 64) * cdiv(m.max_dr, 64);
  const hipError_t e = launch_env_tile(p1, t1 < 512 ? 1 : 0, m.n_par, m.max_dl, 2 * m.max_dr, s);
  return e != hipSuccess ? e : launch_env_tile(p2, t2 < 512 ? 1 : 0, m.n_chi, m.max_dr, m.max_dr, s);
}

template <typename L>
hipError_t env_merged_split(const EnvMerged& m, hipStream_t s) {
  const EnvG1P<float> p1 = env_p1<float>(m);
  const EnvG2P<float> p2 = env_p2<float>(m);
  const hipError_t e = launch_cgemm_split<L, 64, 64>(p1, m.n_par, m.max_dl, 2 * m.max_dr, s);
  return e != hipSuccess ? e : launch_cgemm_split<L, 64, 64>(p2, m.n_chi, m.max_dr, m.max_dr, s);
}

hipError_t launch_env_merged(const EnvMerged& m, int prec, hipStream_t s) {
  switch (prec) {
    case 0: return env_merged_t<double>(m, s);
    case 1: return env_merged_t<float>(m, s);
    case 2: return env_merged_split<__bf16>(m, s);
    case 3: return env_merged_split<_Float16>(m, s);
    default: return hipErrorInvalidValue;
  }
}

// A whole update L' = sum_s A^{s+} (phase X^{s^flip}), X = L [A^0 | A^1], of one
// child per workgroup, X in LDS, operands straight from L2.  Small dims are
// bound by launches and by the latency of a staged K loop (6 + 12 us for the
// two GEMMs at D = 32).  X is recomputed for every child of a parent, which is
// cheaper than a launch and a round trip of X up to dims of 32, whether the launch
// has fewer children than the chip has compute units or fills it many times over,
// and with up to four children per parent.  Whole expectations in c128 ms, the two
// GEMMs / this kernel: 16 qubits D = 8, 16 strings 0.19 / 0.15, 20,000 (7,600
// children a launch) 1.71 / 0.60; D = 32, 1,000 strings 0.63 / 0.34, 20,000 5.03 /
// 2.38; every string on seven sites (three children per parent) 0.27 / 0.24.
// Above: D = 48 0.25 / 0.34 (16 strings) and 8.18 / 7.81 (20,000), D = 64 0.27 / 0.47
// and 11.3 / 20.5.  Per element the same operations in the same order as
// cgemm_kernel on EnvG1P and EnvG2P.
template <typename T>
__global__ __launch_bounds__(256) void env_small_kernel(const EnvSeg* segs, int n_segs) {
  using C2 = typename cplx_of<T>::type;
  using Acc = typename acc_of<T>::type;
  extern __shared__ double2 env_lds[];
  C2* X = (C2*)env_lds;  // [dl][2 dr + 1]
  const int item = blockIdx.x;
  int base;
  const EnvSeg g = segs[find_segment<&EnvSeg::chi_end>(segs, n_segs, item, base)];
  const EnvChild<C2> ch = ((const EnvChild<C2>*)g.chi)[item - base];
  const int dl = g.dl, dr = g.dr, ldx = 2 * dr + 1;
  const C2* site = (const C2*)g.site;
  const int sk = g.trans ? 1 : dr, sj = g.trans ? dl : 1;  // site[s][k][j]
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const int tl = (dl + 15) / 16, tr = (dr + 15) / 16;
  for (int t = wv; t < tl * tr; t += 4) {
    const int i0 = (t / tr) * 16, j0 = (t % tr) * 16;
    const C2* pa = ch.l + (size_t)min(i0 + lr, dl - 1) * dl;
    const C2* pb = site + (size_t)min(j0 + lr, dr - 1) * sj;
    Acc re[1][2], im[1][2];
    wave_gemm<T, 1, 2>(
        re, im, dl, [&](int, int k) { return pa[k]; },
        [&](int s, int k) { return pb[(size_t)s * dl * dr + (size_t)k * sk]; });
    const int j = j0 + lr;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = i0 + acc_row<T>(lk, v);
        if (i < dl && j < dr) {
          C2 o;
          o.x = re[0][s][v];
          o.y = im[0][s][v];
          X[(size_t)i * ldx + s * dr + j] = o;
        }
      }
  }
  __syncthreads();
  const int flip = (ch.letter == 1 || ch.letter == 2) ? 1 : 0;
  for (int t = wv; t < tr * tr; t += 4) {
    const int i0 = (t / tr) * 16, j0 = (t % tr) * 16;
    const C2* pa = site + (size_t)min(i0 + lr, dr - 1) * sj;
    const C2* pb = X + min(j0 + lr, dr - 1);
    Acc re[1][1], im[1][1];
    wave_gemm<T, 1, 1>(
        re, im, 2 * dl,
        [&](int, int k) {
          const int s = k >= dl, a = k - s * dl;
          C2 v = pa[(size_t)s * dl * dr + (size_t)a * sk];
          v.y = -v.y;
          return v;
        },
        [&](int, int k) {
          const int s = k >= dl, a = k - s * dl;
          const C2 v = pb[(size_t)a * ldx + (s ^ flip) * dr];
          C2 o = v;
          if (ch.letter == 2) {  // Y: s=0 -> -i X^1, s=1 -> +i X^0
            o.x = s == 0 ? v.y : -v.y;
            o.y = s == 0 ? -v.x : v.x;
          } else if (ch.letter == 3 && s == 1) {
            o.x = -v.x;
            o.y = -v.y;
          }
          return o;
        });
    const int j = j0 + lr;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = i0 + acc_row<T>(lk, v);
      if (i < dr && j < dr) {
        C2 o;
        o.x = re[0][0][v];
        o.y = im[0][0][v];
        ch.out[(size_t)i * dr + j] = o;
      }
    }
  }
}

hipError_t configure_env_small() {
  const int bytes = kEnvSmall * (2 * kEnvSmall + 1) * (int)sizeof(double2);
  const hipError_t e = hipFuncSetAttribute((const void*)env_small_kernel<double>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  return e != hipSuccess ? e
                         : hipFuncSetAttribute((const void*)env_small_kernel<float>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, bytes / 2);
}

hipError_t launch_env_small(const EnvMerged& m, int prec, hipStream_t s) {
  if (m.n_chi <= 0) return hipSuccess;
  if (m.max_dl > kEnvSmall || m.max_dr > kEnvSmall || prec > 1) return hipErrorInvalidValue;
  const size_t el = (size_t)m.max_dl * (2 * m.max_dr + 1);
  if (prec == 0)
    hipLaunchKernelGGL(env_small_kernel<double>, dim3(m.n_chi), dim3(256), el * sizeof(double2), s, m.segs, m.n_segs);
  else
    hipLaunchKernelGGL(env_small_kernel<float>, dim3(m.n_chi), dim3(256), el * sizeof(float2), s, m.segs, m.n_segs);
  return hipGetLastError();
}

// Site tensor in the environment precision (fwd, may be null) and its
// per-letter transpose tr[s][beta][alpha] = B[s][alpha][beta], which turns the
// right update R' = sum sigma B^{s'} R B^{s+} into the left form on R^T.
template <typename C2>
__global__ void site_prepare_kernel(const double2* site, C2* fwd, C2* tr, int dl, int dr) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  const int per = dl * dr;
  if (idx >= 2 * per) return;
  const int s = idx / per;
  const int rem = idx - s * per;
  const int a = rem / dr, b = rem - (rem / dr) * dr;
  const double2 v = site[idx];
  C2 o;
  o.x = v.x;
  o.y = v.y;
  if (fwd) fwd[idx] = o;
  tr[(size_t)s * per + (size_t)b * dl + a] = o;
}

hipError_t launch_site_prepare(const double2* site, void* out_fwd, void* out_tr, int dl, int dr,
                               int elem_bytes, hipStream_t s) {
  const int blocks = cdiv(2LL * dl * dr, 256);
  if (elem_bytes == 16)
    hipLaunchKernelGGL(site_prepare_kernel<double2>, dim3(blocks), dim3(256), 0, s, site,
                       (double2*)out_fwd, (double2*)out_tr, dl, dr);
  else
    hipLaunchKernelGGL(site_prepare_kernel<float2>, dim3(blocks), dim3(256), 0, s, site,
                       (float2*)out_fwd, (float2*)out_tr, dl, dr);
  return hipGetLastError();
}

// Roots of the two tries at one bond: diag(lambda^2) (Eq. expec1/expec2) and
// the identity (right boundary in right-canonical form, Eq. rc).
template <typename C2>
__global__ void roots_kernel(const double* lam, C2* lroot, C2* rroot, int d) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= d * d) return;
  const int i = idx / d, j = idx - (idx / d) * d;
  C2 z;
  z.x = 0;
  z.y = 0;
  C2 lv = z, rv = z;
  if (i == j) {
    lv.x = lam[i] * lam[i];
    rv.x = 1;
  }
  if (lroot) lroot[idx] = lv;
  if (rroot) rroot[idx] = rv;
}

hipError_t launch_roots(const double* lam, void* lroot, void* rroot, int d, int elem_bytes,
                        hipStream_t s) {
  const int blocks = cdiv((long long)d * d, 256);
  if (elem_bytes == 16)
    hipLaunchKernelGGL(roots_kernel<double2>, dim3(blocks), dim3(256), 0, s, lam, (double2*)lroot,
                       (double2*)rroot, d);
  else
    hipLaunchKernelGGL(roots_kernel<float2>, dim3(blocks), dim3(256), 0, s, lam, (float2*)lroot,
                       (float2*)rroot, d);
  return hipGetLastError();
}

// FP64 environment -> a root slot in the environment precision.
template <typename C2>
__global__ void root_copy_kernel(const double2* src, C2* dst, size_t count) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < count) {
    C2 v;
    v.x = src[i].x;
    v.y = src[i].y;
    dst[i] = v;
  }
}

hipError_t launch_root_copy(const double2* src, void* dst, size_t count, int elem_bytes, hipStream_t s) {
  if (count == 0) return hipSuccess;
  const int blocks = cdiv((long long)count, 256);
  if (elem_bytes == 16)
    hipLaunchKernelGGL(root_copy_kernel<double2>, dim3(blocks), dim3(256), 0, s, src, (double2*)dst, count);
  else
    hipLaunchKernelGGL(root_copy_kernel<float2>, dim3(blocks), dim3(256), 0, s, src, (float2*)dst, count);
  return hipGetLastError();
}

// Lists of the two kernels above in one launch each (several states'
// set-up): block row y takes item y, 256 elements per block along x.
template <typename C2>
__global__ void site_prepare_list_kernel(const PrepItem* items) {
  const PrepItem it = items[blockIdx.y];
  const int idx = blockIdx.x * 256 + threadIdx.x;
  const int per = it.dl * it.dr;
  if (idx >= 2 * per) return;
  const int s = idx / per;
  const int rem = idx - s * per;
  const int a = rem / it.dr, b = rem - (rem / it.dr) * it.dr;
  const double2 v = it.site[idx];
  C2 o;
  o.x = v.x;
  o.y = v.y;
  if (it.fwd) ((C2*)it.fwd)[idx] = o;
  ((C2*)it.tr)[(size_t)s * per + (size_t)b * it.dl + a] = o;
}

hipError_t launch_site_prepare_list(const PrepItem* items, int count, int max_elems, int elem_bytes,
                                    hipStream_t s) {
  if (count <= 0 || max_elems <= 0) return hipSuccess;
  if (count > 65535) return hipErrorInvalidValue;
  const dim3 grid(cdiv((long long)max_elems, 256), count);
  if (elem_bytes == 16)
    hipLaunchKernelGGL(site_prepare_list_kernel<double2>, grid, dim3(256), 0, s, items);
  else
    hipLaunchKernelGGL(site_prepare_list_kernel<float2>, grid, dim3(256), 0, s, items);
  return hipGetLastError();
}

template <typename C2>
__global__ void root_copy_list_kernel(const CopyItem* items) {
  const CopyItem it = items[blockIdx.y];
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i < it.count) {
    C2 v;
    v.x = it.src[i].x;
    v.y = it.src[i].y;
    ((C2*)it.dst)[i] = v;
  }
}

hipError_t launch_root_copy_list(const CopyItem* items, int count, long long max_count, int elem_bytes,
                                 hipStream_t s) {
  if (count <= 0 || max_count <= 0) return hipSuccess;
  if (count > 65535) return hipErrorInvalidValue;
  const dim3 grid(cdiv(max_count, 256), count);
  if (elem_bytes == 16)
    hipLaunchKernelGGL(root_copy_list_kernel<double2>, grid, dim3(256), 0, s, items);
  else
    hipLaunchKernelGGL(root_copy_list_kernel<float2>, grid, dim3(256), 0, s, items);
  return hipGetLastError();
}

// Closing traces: Tr(L_a R_b) = sum_{xy} L_a[x][y] R_b[y][x] = sum_x L_a[x] R^T_b[x]
// with right environments stored transposed; computed in FP64, real part
// only, for the 64x64 tiles of (prefix, suffix) pairs that some string needs.
template <typename C2>
struct GramTileP {
  using T = double;
  struct Ctx {
    const void* const* lptr;
    const void* const* rptr;
    double* g;
    int m, n, k, ldg;
  };
  using RowA = const C2*;
  using ColB = const C2*;
  static constexpr bool A_CONTIG_K = true, B_CONTIG_N = false, REAL_ONLY = true;
  const GramItem* items;
  const GramTile* tiles;
  __device__ Ctx context(int i) const {
    const GramTile t = tiles[i];
    const GramItem b = items[t.item];
    return Ctx{b.lptr + t.r0, b.rptr + t.c0, b.g + (size_t)t.r0 * b.nr + t.c0,
               min(64, b.nl - t.r0), min(64, b.nr - t.c0), b.kdim, b.nr};
  }
  __device__ static void dims(const Ctx& c, int& M, int& N, int& K) {
    M = c.m;
    N = c.n;
    K = c.k;
  }
  __device__ static RowA rowA(const Ctx& c, int i) { return (const C2*)c.lptr[i]; }
  __device__ static ColB colB(const Ctx& c, int j) { return (const C2*)c.rptr[j]; }
  __device__ static double2 loadA(const Ctx&, RowA r, int, int k) {
    const C2 v = r[k];
    return make_double2((double)v.x, (double)v.y);
  }
  __device__ static double2 loadB(const Ctx&, ColB b, int k, int) {
    const C2 v = b[k];
    return make_double2((double)v.x, (double)v.y);
  }
  __device__ static void store(const Ctx& c, int i, int j, double re, double) {
    c.g[(size_t)i * c.ldg + j] = re;
  }
};

// Split-K form: item i = split * n_tiles + tile sums the K range of its split
// (K / splits rounded up to 16) into part[i] (64 x 64, row-major); gram_reduce
// then adds the splits in a fixed order, so the result does not depend on
// scheduling.  Long traces (K = D^2 up to 262144) are split so that a
// launch has enough workgroups to fill the chip.
template <typename C2>
struct GramSplitP {
  using T = double;
  struct Ctx {
    const void* const* lptr;
    const void* const* rptr;
    double* part;
    int m, n, k0, k;
  };
  using RowA = const C2*;
  using ColB = const C2*;
  static constexpr bool A_CONTIG_K = true, B_CONTIG_N = false, REAL_ONLY = true;
  const GramItem* items;
  const GramTile* tiles;
  double* part;
  int n_tiles, splits;
  __device__ Ctx context(int i) const {
    const int tile = i % n_tiles, sp = i / n_tiles;
    const GramTile t = tiles[tile];
    const GramItem b = items[t.item];
    const int chunk = ((b.kdim + splits - 1) / splits + 15) & ~15;
    const int k0 = min(b.kdim, sp * chunk);
    const int k1 = min(b.kdim, k0 + chunk);
    return Ctx{b.lptr + t.r0, b.rptr + t.c0, part + (size_t)i * 4096, min(64, b.nl - t.r0),
               min(64, b.nr - t.c0), k0, k1 - k0};
  }
  __device__ static void dims(const Ctx& c, int& M, int& N, int& K) {
    M = c.m;
    N = c.n;
    K = c.k;
  }
  __device__ static RowA rowA(const Ctx& c, int i) { return (const C2*)c.lptr[i] + c.k0; }
  __device__ static ColB colB(const Ctx& c, int j) { return (const C2*)c.rptr[j] + c.k0; }
  __device__ static double2 loadA(const Ctx&, RowA r, int, int k) {
    const C2 v = r[k];
    return make_double2((double)v.x, (double)v.y);
  }
  __device__ static double2 loadB(const Ctx&, ColB b, int k, int) {
    const C2 v = b[k];
    return make_double2((double)v.x, (double)v.y);
  }
  __device__ static void store(const Ctx& c, int i, int j, double re, double) { c.part[i * 64 + j] = re; }
};

__global__ void gram_reduce_kernel(const GramItem* items, const GramTile* tiles, const double* part,
                                   int n_tiles, int splits) {
  const int tile = blockIdx.x;
  const GramTile t = tiles[tile];
  const GramItem b = items[t.item];
  const int m = min(64, b.nl - t.r0), n = min(64, b.nr - t.c0);
  for (int e = threadIdx.x; e < 4096; e += blockDim.x) {
    const int i = e >> 6, j = e & 63;
    if (i >= m || j >= n) continue;
    double acc = 0.0;
    for (int sp = 0; sp < splits; ++sp) acc += part[((size_t)sp * n_tiles + tile) * 4096 + e];
    b.g[(size_t)(t.r0 + i) * b.nr + t.c0 + j] = acc;
  }
}

int gram_splits(int max_kdim) { return max_kdim >= 32768 ? 8 : (max_kdim >= 8192 ? 4 : 1); }

hipError_t launch_gram(const GramItem* items_dev, const GramTile* tiles_dev, int n_tiles, int elem_bytes,
                       double* part, int splits, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  if (splits <= 1 || !part) {
    if (elem_bytes == 16) {
      GramTileP<double2> p{items_dev, tiles_dev};
      return launch_cgemm<64, 64, 16>(p, n_tiles, 64, 64, s);
    }
    GramTileP<float2> p{items_dev, tiles_dev};
    return launch_cgemm<64, 64, 16>(p, n_tiles, 64, 64, s);
  }
  hipError_t e;
  if (elem_bytes == 16) {
    GramSplitP<double2> p{items_dev, tiles_dev, part, n_tiles, splits};
    e = launch_cgemm<64, 64, 16>(p, n_tiles * splits, 64, 64, s);
  } else {
    GramSplitP<float2> p{items_dev, tiles_dev, part, n_tiles, splits};
    e = launch_cgemm<64, 64, 16>(p, n_tiles * splits, 64, 64, s);
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(gram_reduce_kernel, dim3(n_tiles), dim3(256), 0, s, items_dev, tiles_dev, part, n_tiles,
                     splits);
  return hipGetLastError();
}

// Closing traces pair by pair, for bonds whose needed pairs fill the tiles
// sparsely: one workgroup per left environment and up to kGramGroup right ones,
// FP64 accumulation in a fixed order (thread, wave, workgroup).  Bound by
// reading the environments (one right environment per pair, the left one
// shared).
template <typename C2>
__global__ __launch_bounds__(256) void gram_pairs_kernel(const GramGroup* groups, const GramPair* pairs) {
  __shared__ double part[4][kGramGroup];
  const GramGroup gr = groups[blockIdx.x];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const C2* l = (const C2*)gr.l;
  const C2* r[kGramGroup];
#pragma unroll
  for (int p = 0; p < kGramGroup; ++p) r[p] = (const C2*)pairs[gr.first + min(p, gr.count - 1)].r;
  double acc[kGramGroup];
#pragma unroll
  for (int p = 0; p < kGramGroup; ++p) acc[p] = 0.0;
  auto run = [&](auto cnt) {
    constexpr int C = decltype(cnt)::value;
    constexpr int U = 4;  // elements in flight per thread and environment
    int e = tid;
    for (; e + (U - 1) * 256 < gr.kdim; e += U * 256) {
      C2 a[U], b[C][U];
#pragma unroll
      for (int u = 0; u < U; ++u) a[u] = l[e + u * 256];
#pragma unroll
      for (int p = 0; p < C; ++p)
#pragma unroll
        for (int u = 0; u < U; ++u) b[p][u] = r[p][e + u * 256];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int p = 0; p < C; ++p)
          acc[p] = fma(-(double)a[u].y, (double)b[p][u].y, fma((double)a[u].x, (double)b[p][u].x, acc[p]));
    }
    for (; e < gr.kdim; e += 256) {
      const C2 a = l[e];
#pragma unroll
      for (int p = 0; p < C; ++p) {
        const C2 b = r[p][e];
        acc[p] = fma(-(double)a.y, (double)b.y, fma((double)a.x, (double)b.x, acc[p]));
      }
    }
  };
  if (gr.count == 1) run(std::integral_constant<int, 1>{});
  else if (gr.count == 2) run(std::integral_constant<int, 2>{});
  else run(std::integral_constant<int, kGramGroup>{});
#pragma unroll
  for (int p = 0; p < kGramGroup; ++p) {
    const double s = wave_sum(acc[p]);
    if (lane == 0) part[wv][p] = s;
  }
  __syncthreads();
  if (tid < gr.count) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < 4; ++w) s += part[w][tid];
    *pairs[gr.first + tid].g = s;
  }
}

// Tiles take the matrix cores' time for all of their 4096 pairs, 22.5 us of the
// chip per 65536 elements in c128 and 28 us in c64 (converted on the way), and,
// however few they are, that of one tile's K range on one workgroup, 0.1 and
// 0.2 us an element (a third of it also where they are many).  Pairs stream their
// environments (the left one once per group) at about 7.5 TB/s, after 5 us.  All bonds' tiles are one launch and all
// pairs another, so the choice is made for all bonds together: the k bonds that
// gain most as tiles are tiles, for the k of least total.  Closes of molecular
// sums in ms, as tiles / as pairs / by this rule / chosen bond by bond, where the
// few tiles of every bond seemed bound by one workgroup's K range:
//   40 qubits D = 128 c128,  16,385 strings  1.53   0.89  0.89   0.90
//                           200,001          2.16   8.47  2.19   4.20
//   50 qubits D = 256 c128,  32,769         12.6    7.20  7.17   7.18
//                           262,144         11.9   46.2  11.8   13.9
//   50 qubits D = 256 c64,   32,769         14.8    3.44  3.46   3.46
//                           262,144         14.1   23.9  14.3   15.6
std::vector<char> gram_choose(const std::vector<GramWork>& bonds, int elem_bytes) {
  const int n = (int)bonds.size();
  const double per_tile = elem_bytes == 16 ? 22.5 : 28.0, per_k = elem_bytes == 16 ? 0.1 : 0.2;
  std::vector<double> pair_us(n), tile_us(n);
  double pairs = 0.0;
  for (int i = 0; i < n; ++i) {
    pair_us[i] = (double)(bonds[i].pairs + bonds[i].groups) * bonds[i].kdim * elem_bytes / 7.5e6;
    tile_us[i] = (double)bonds[i].tiles * bonds[i].kdim * per_tile / 65536;
    pairs += pair_us[i];
  }
  std::vector<int> order(n);
  for (int i = 0; i < n; ++i) order[i] = i;
  std::stable_sort(order.begin(), order.end(),
                   [&](int a, int b) { return pair_us[a] - tile_us[a] > pair_us[b] - tile_us[b]; });
  int best = 0, longest = 0;
  double least = 5.0 + pairs, tiles = 0.0;
  for (int k = 1; k <= n; ++k) {
    const int i = order[k - 1];
    tiles += tile_us[i];
    pairs -= pair_us[i];
    longest = std::max(longest, bonds[i].kdim);
    const double one = per_k * longest / gram_splits(longest);
    const double cost = std::max(one, tiles + 0.3 * one) + (k < n ? 5.0 + pairs : 0.0);
    if (cost < least) {
      least = cost;
      best = k;
    }
  }
  std::vector<char> as_pairs(n, 1);
  for (int k = 0; k < best; ++k) as_pairs[order[k]] = 0;
  return as_pairs;
}

hipError_t launch_gram_pairs(const GramGroup* groups_dev, const GramPair* pairs_dev, int groups, int elem_bytes,
                             hipStream_t s) {
  if (groups <= 0) return hipSuccess;
  if (elem_bytes == 16)
    hipLaunchKernelGGL(gram_pairs_kernel<double2>, dim3(groups), dim3(256), 0, s, groups_dev, pairs_dev);
  else
    hipLaunchKernelGGL(gram_pairs_kernel<float2>, dim3(groups), dim3(256), 0, s, groups_dev, pairs_dev);
  return hipGetLastError();
}

// <P_k> = closing trace / <psi|psi> (nrm null: unit norm)
__global__ void gather_kernel(const double* g, const int64_t* gidx, const double2* nrm, double* per_term,
                              int64_t n) {
  const int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x;
  if (i < n) per_term[i] = nrm ? g[gidx[i]] / nrm->x : g[gidx[i]];
}

hipError_t launch_gather(const double* g, const int64_t* gidx, const double2* nrm, double* per_term,
                         int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(gather_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, g, gidx, nrm,
                     per_term, n);
  return hipGetLastError();
}

// E = sum_k c_k <P_k>: each thread a contiguous chunk with error-free
// transformations (TwoProduct by fma, TwoSum), then a fixed-shape tree of
// double-double additions -- the result depends only on the string order.
__device__ __forceinline__ void two_sum(double a, double b, double& s, double& e) {
  s = a + b;
  const double bb = s - a;
  e = (a - (s - bb)) + (b - bb);
}

__global__ __launch_bounds__(1024) void energy_kernel(const double* per_term, const double* coeffs,
                                                      int64_t n, double* out) {
  __shared__ double hs[1024], ls[1024];
  const int64_t chunk = (n + 1023) / 1024;
  const int64_t lo = threadIdx.x * chunk;
  const int64_t hi = lo + chunk < n ? lo + chunk : n;
  double s = 0.0, c = 0.0;
  for (int64_t i = lo; i < hi; ++i) {
    const double p = coeffs[i] * per_term[i];
    const double pe = fma(coeffs[i], per_term[i], -p);
    double t, e;
    two_sum(s, p, t, e);
    s = t;
    c += e + pe;
  }
  hs[threadIdx.x] = s;
  ls[threadIdx.x] = c;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      double t, e;
      two_sum(hs[threadIdx.x], hs[threadIdx.x + w], t, e);
      hs[threadIdx.x] = t;
      ls[threadIdx.x] = ls[threadIdx.x] + ls[threadIdx.x + w] + e;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {  // the compensated pair (sum, error); the value is their sum
    out[0] = hs[0];
    out[1] = ls[0];
  }
}

// Several compensated pairs (hi_i, lo_i), i < n, added in index order with the
// same error-free transformations: out[0] = sum, out[1] = error.
__global__ void pair_sum_kernel(const double* pairs, int n, double* out) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  double s = 0.0, c = 0.0;
  for (int i = 0; i < n; ++i) {
    double t, e;
    two_sum(s, pairs[2 * i], t, e);
    s = t;
    c += e + pairs[2 * i + 1];
  }
  out[0] = s;
  out[1] = c;
}

hipError_t launch_pair_sum(const double* pairs, int n, double* out, hipStream_t s) {
  hipLaunchKernelGGL(pair_sum_kernel, dim3(1), dim3(64), 0, s, pairs, n, out);
  return hipGetLastError();
}

// out[r] = sum_{i in row r} vals[i] <P_{cols[i]}>, one thread per row, with
// the same error-free transformations as the energy (result depends only on
// the order of the row's entries).
__global__ void rows_kernel(const double* per_term, const int64_t* row_ptr, const int64_t* cols,
                           const double* vals, int64_t n_rows, double* out) {
  const int64_t r = blockIdx.x * (int64_t)256 + threadIdx.x;
  if (r >= n_rows) return;
  double s = 0.0, c = 0.0;
  for (int64_t i = row_ptr[r]; i < row_ptr[r + 1]; ++i) {
    const double p = vals[i] * per_term[cols[i]];
    const double pe = fma(vals[i], per_term[cols[i]], -p);
    double t, e;
    two_sum(s, p, t, e);
    s = t;
    c += e + pe;
  }
  out[r] = s + c;
}

hipError_t launch_rows(const double* per_term, const int64_t* row_ptr, const int64_t* cols, const double* vals,
                       int64_t n_rows, double* out, hipStream_t s) {
  if (n_rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(rows_kernel, dim3((unsigned)((n_rows + 255) / 256)), dim3(256), 0, s, per_term, row_ptr,
                     cols, vals, n_rows, out);
  return hipGetLastError();
}

hipError_t launch_energy(const double* per_term, const double* coeffs, int64_t n, double* out,
                         hipStream_t s) {
  hipLaunchKernelGGL(energy_kernel, dim3(1), dim3(1024), 0, s, per_term, coeffs, n, out);
  return hipGetLastError();
}

// One 16x16x4 MFMA of known operands in FP64 (out[0..255]) and FP32
// (out[256..511]), written back through the accumulator layout the GEMMs use.
__global__ void selftest_mfma_kernel(double* out) {
  const int l = threadIdx.x;
  const int r = l & 15, k = l >> 4;
  const double a = 1.0 + r + 0.5 * k;            // A[r][k]
  const double b = 1.0 + 0.25 * k - 0.125 * r;   // B[k][r]
  d4_t acc = {0.0, 0.0, 0.0, 0.0};
  acc = mfma_16x16x4(a, b, acc);
  f4_t facc = {0.f, 0.f, 0.f, 0.f};
  facc = mfma_16x16x4((float)a, (float)b, facc);
  // 16x16x32: A[i][kk] = ((i + 2 kk) mod 7) - 3, B[kk][j] = ((3 kk + j) mod 5) - 2 (exact in 16 bits)
  bf16x8_t ab, bb;
  f16x8_t ah, bh;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int kk = frag32_k(l, j);
    const float av = (float)(((r + 2 * kk) % 7) - 3), bv = (float)(((3 * kk + r) % 5) - 2);
    ab[j] = (__bf16)av;
    bb[j] = (__bf16)bv;
    ah[j] = (_Float16)av;
    bh[j] = (_Float16)bv;
  }
  f4_t c16 = {0.f, 0.f, 0.f, 0.f}, d16 = {0.f, 0.f, 0.f, 0.f};
  c16 = split_traits<__bf16>::mfma(ab, bb, c16);
  d16 = split_traits<_Float16>::mfma(ah, bh, d16);
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    out[acc_row<double>(k, v) * 16 + r] = acc[v];
    out[256 + acc_row<float>(k, v) * 16 + r] = (double)facc[v];
    out[512 + acc_row<float>(k, v) * 16 + r] = (double)c16[v];
    out[768 + acc_row<float>(k, v) * 16 + r] = (double)d16[v];
  }
}

hipError_t launch_selftest_mfma(double* out, hipStream_t s) {
  hipLaunchKernelGGL(selftest_mfma_kernel, dim3(1), dim3(64), 0, s, out);
  return hipGetLastError();
}

}  // namespace mps
