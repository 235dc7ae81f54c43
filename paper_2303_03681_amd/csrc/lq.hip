// LQ preconditioning of the batched gate SVDs (Eq. svd with Algorithm 1).
//
// Algorithm 1 applied to the rows of C~ directly needs up to 23 sweeps on the
// central bonds of a saturated state: the rows carry the graded lambda of
// Eq. (C~), and the few smallest directions keep relative inner products near
// one for ten sweeps after the others have converged.  Two LQ factorisations
// (rows sorted by norm) move the grading to where the rotations see a nearly
// diagonal matrix:
//
//   P C~ = L1 Q1,   L1^+ = L2 Q2,   Algorithm 1 on the rows of L2^+ :
//   J L2^+ = Sigma Z,  and  V^+ = Z Q1.
//
// A tall C~ (more rows than columns) is first replaced by the triangular
// factor of its columns, C~^+ = L0 Q0 -> L0^+ (square, the same right vectors),
// so that every row of every factorisation is a step: the leading rows of a
// tall matrix need not span its row space.
//
// (The rows of L2^+ have the Gram matrix of the columns of L2; X = Z^+ are the
// left singular vectors of L1^+, that is the right ones of L1.)  Sweeps until
// no rotation, measured on captured 512 x 512 C~ of a 30-qubit D = 256
// brickwork state: 21-23 without, 12-13 after one, 9-10 after two
// factorisations; 128 x 128 of a UCCSD chain: 18-31 without, 6-8 after two.
//
// The factorisations are modified Gram-Schmidt over blocks of rows (the
// factor L of MGS is as accurate as Householder's): lq_panel_kernel
// orthonormalises one block of every matrix, lq_update_kernel takes the
// block's components out of all later rows.  The rows of Z Q1 are orthonormal
// to eps sigma_1 / sigma_p only (the loss of MGS in Q1), so they go through
// the same two kernels once more in descending order of sigma, which leaves
// the leading directions untouched and leaves nothing of a row that depends on
// earlier ones to rounding (kDependent).
//
// What bounds it: the panel is a serial chain of LQB steps (norm, broadcast
// through LDS, dot products, update) on one workgroup per matrix; the update
// is FP64 vector work on all compute units, its rows read and written once
// per block.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "gemm_core.h"
#include "internal.h"
#include "lq_ops.h"
#include "wave_ops.h"

namespace mps {

namespace {

inline int cdiv(long long a, long long b) { return (int)((a + b - 1) / b); }

// Row i of the matrix (in processing order).
__device__ __forceinline__ double2* lq_row(const LqItem& it, int i) {
  return it.w + (size_t)(it.order ? it.order[i] : i) * it.m;
}

__device__ __forceinline__ int lq_rows(const LqItem& it) {
  return it.k_dev ? min(it.n, *it.k_dev) : it.n;
}

// One row, lane + 64 k to element k: every lane loads from inside the row (the
// index clamped to its end) and zeroes what lies outside it.
template <int E>
__device__ __forceinline__ void load_row(double2 (&x)[E], const double2* src, bool valid, int m, int lane) {
  const gdvec2* g = (const gdvec2*)src;
#pragma unroll
  for (int k = 0; k < E; ++k) {
    const int e = lane + 64 * k;
    const dvec2 v = g[e < m ? e : m - 1];
    const bool keep = valid && e < m;
    x[k] = make_double2(keep ? v.x : 0.0, keep ? v.y : 0.0);
  }
}

}  // namespace

// Squared norms of the rows of every matrix, one wave per row.
__global__ __launch_bounds__(256) void row_norm_kernel(const LqItem* items, int per_item) {
  const int item = blockIdx.x / per_item;
  const LqItem it = items[item];
  const int row = (blockIdx.x - item * per_item) * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= it.n) return;
  const double2* w = it.w + (size_t)row * it.m;
  double s = 0.0;
  for (int e = lane; e < it.m; e += 64) s = norm_acc(w[e], s);
  s = wave_sum(s);
  if (lane == 0) it.norm2[row] = s;
}

hipError_t launch_row_norm(const LqItem* items_dev, int items, int max_rows, hipStream_t s) {
  if (items <= 0 || max_rows <= 0) return hipSuccess;
  const int per = cdiv(max_rows, 4);
  hipLaunchKernelGGL(row_norm_kernel, dim3(items * per), dim3(256), 0, s, items_dev, per);
  return hipGetLastError();
}

// Row order by descending norm (ties by index), one workgroup per matrix.
__global__ __launch_bounds__(1024) void lq_order_kernel(const LqItem* items) {
  __shared__ double key[1024];
  const LqItem it = items[blockIdx.x];
  const int i = threadIdx.x, n = it.n;
  if (i < n) {
    // a NaN sorts first, so that every position is written
    const double v = it.norm2[i];
    key[i] = v == v ? v : INFINITY;
  }
  __syncthreads();
  if (i >= n) return;
  const double mine = key[i];
  int r = 0;
  for (int j = 0; j < n; ++j) r += (key[j] > mine) || (key[j] == mine && j < i);
  it.order_out[r] = i;
}

hipError_t launch_lq_order(const LqItem* items_dev, int items, hipStream_t s) {
  if (items <= 0) return hipSuccess;
  hipLaunchKernelGGL(lq_order_kernel, dim3(items), dim3(1024), 0, s, items_dev);
  return hipGetLastError();
}

// Modified Gram-Schmidt inside block `panel` (LQB rows) of every matrix, one
// workgroup of NW waves per matrix.  Row s of the factor gets its diagonal and
// in-block entries, and zeros before the diagonal.
template <int E, int NW, int RPW>
__global__ __launch_bounds__(NW * 64) void lq_panel_kernel(const LqItem* items, int panel) {
  constexpr int LQB = NW * RPW;
  __shared__ double2 q_lds[2][64 * E];
  const LqItem it = items[blockIdx.x];
  const int n = lq_rows(it), m = it.m;
  const int s0 = panel * LQB;
  if (s0 >= n) return;
  const int nb = min(LQB, n - s0);
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double2 x[RPW][E];
#pragma unroll
  for (int a = 0; a < RPW; ++a) {
    const int u = a * NW + wv;
    load_row<E>(x[a], lq_row(it, s0 + min(u, nb - 1)), u < nb, m, lane);
  }
  const int half = m / 2;
  mgs_rows<E, NW, RPW>(
      x, nb, &q_lds[0][0], it.out ? kDependent : 0.0,
      [&](int t, double r) {
        if (it.r) it.r[(size_t)(s0 + t) * it.n + s0 + t] = make_double2(r, 0.0);
      },
      [&](int t, const double2* q) {  // the finished row, and the factor's zeros before the diagonal
        gdvec2* dst = (gdvec2*)lq_row(it, s0 + t);
        for (int e = threadIdx.x; e < m; e += NW * 64) {
          const double2 v = q[e];
          dst[e] = dvec2{v.x, v.y};
          if (it.out) {  // [s][row][r], the layout of a right site tensor
            const int sb = e >= half ? 1 : 0;
            it.out[((size_t)sb * n + s0 + t) * half + e - sb * half] = v;
          }
        }
        if (it.r)
          for (int i = threadIdx.x; i < s0 + t; i += NW * 64)
            it.r[(size_t)(s0 + t) * it.n + i] = make_double2(0.0, 0.0);
      },
      [&](int t, int u, double re, double im) {
        if (it.r) it.r[(size_t)(s0 + t) * it.n + s0 + u] = make_double2(re, -im);
      });
}

// Takes the components along the rows of block `panel` out of every later row
// (one after the other, so modified Gram-Schmidt across blocks too): four
// waves of RPW rows each, the block's rows staged through LDS QC at a time.
template <int E, int LQB, int RPW>
__global__ __launch_bounds__(256, 2) void lq_update_kernel(const LqItem* items, int panel, int per_item) {
  constexpr int QC = LQB < 64 / E ? LQB : 64 / E;  // 64 KB of rows at a time
  __shared__ double2 q_lds[QC][64 * E];
  const int item = blockIdx.x / per_item;
  const LqItem it = items[item];
  const int n = lq_rows(it), m = it.m;
  const int s0 = panel * LQB;
  if (s0 >= n) return;
  const int nb = min(LQB, n - s0);
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int first = s0 + nb + (blockIdx.x - item * per_item) * 4 * RPW;
  if (first >= n) return;
  const int i0 = first + wv * RPW;
  double2 x[RPW][E];
#pragma unroll
  for (int a = 0; a < RPW; ++a) {
    load_row<E>(x[a], lq_row(it, min(i0 + a, n - 1)), i0 + a < n, m, lane);
  }
  for (int t0 = 0; t0 < nb; t0 += QC) {
    const int tc = min(QC, nb - t0);
    __syncthreads();
    for (int t = wv; t < tc; t += 4) {
      double2 v[E];
      load_row<E>(v, lq_row(it, s0 + t0 + t), true, m, lane);
#pragma unroll
      for (int k = 0; k < E; ++k) q_lds[t][lane + 64 * k] = v[k];
    }
    __syncthreads();
    for (int t = 0; t < tc; ++t) {
      double2 q[E];
#pragma unroll
      for (int k = 0; k < E; ++k) q[k] = q_lds[t][lane + 64 * k];
      double c[2 * RPW];
#pragma unroll
      for (int a = 0; a < RPW; ++a) {
        c[2 * a] = c[2 * a + 1] = 0.0;
#pragma unroll
        for (int k = 0; k < E; ++k) dot_acc(q[k], x[a][k], c[2 * a], c[2 * a + 1]);
      }
      wave_sum_scalar<2 * RPW>(c, lane);
#pragma unroll
      for (int a = 0; a < RPW; ++a) {
#pragma unroll
        for (int k = 0; k < E; ++k) sub_mul(x[a][k], c[2 * a], c[2 * a + 1], q[k]);
        if (it.r && lane == a && i0 + a < n)
          it.r[(size_t)(s0 + t0 + t) * it.n + i0 + a] = make_double2(c[2 * a], -c[2 * a + 1]);
      }
    }
  }
#pragma unroll
  for (int a = 0; a < RPW; ++a) {
    if (i0 + a >= n) continue;
    gdvec2* dst = (gdvec2*)lq_row(it, i0 + a);
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int e = lane + 64 * k;
      if (e < m) dst[e] = dvec2{x[a][k].x, x[a][k].y};
    }
  }
}

namespace {

template <int E, int NW, int RPW, int URPW>
hipError_t launch_lq_e(const LqItem* items_dev, int items, int max_rows, hipStream_t s) {
  constexpr int LQB = NW * RPW;
  for (int p = 0; p * LQB < max_rows; ++p) {
    hipLaunchKernelGGL((lq_panel_kernel<E, NW, RPW>), dim3(items), dim3(NW * 64), 0, s, items_dev, p);
    const int rest = max_rows - (p + 1) * LQB;
    if (rest > 0) {
      const int per = cdiv(rest, 4 * URPW);
      hipLaunchKernelGGL((lq_update_kernel<E, LQB, URPW>), dim3(items * per), dim3(256), 0, s, items_dev, p,
                         per);
    }
  }
  return hipGetLastError();
}

}  // namespace

// LQ factorisation of every matrix (max_rows x max_len the largest): rows
// become Q in place (in processing order), the factor goes to r as L^+.
// Blocks of 16 rows (32 take 74 us a panel at 8 matrices of 512 columns, 16 take 27).
hipError_t launch_lq(const LqItem* items_dev, int items, int max_rows, int max_len, hipStream_t s) {
  if (items <= 0 || max_rows <= 0 || max_len <= 0) return hipSuccess;
  if (max_len <= 128) return launch_lq_e<2, 8, 2, 4>(items_dev, items, max_rows, s);
  if (max_len <= 256) return launch_lq_e<4, 8, 2, 4>(items_dev, items, max_rows, s);
  if (max_len <= 512) return launch_lq_e<8, 8, 2, 4>(items_dev, items, max_rows, s);
  if (max_len <= 1024) return launch_lq_e<16, 8, 2, 2>(items_dev, items, max_rows, s);
  return hipErrorInvalidValue;
}

// w (n x m) = adjoint of r (m x n), 16 x 16 elements per workgroup through LDS.
__global__ __launch_bounds__(256) void lq_adjoint_kernel(const LqItem* items, int per_item, int tiles_m) {
  __shared__ double2 t[16][17];
  const int item = blockIdx.x / per_item;
  const LqItem it = items[item];
  const int b = blockIdx.x - item * per_item;
  const int i0 = (b / tiles_m) * 16, j0 = (b % tiles_m) * 16;  // rows and columns of w
  const int x = threadIdx.x & 15, y = threadIdx.x >> 4;
  if (i0 >= it.n || j0 >= it.m) return;
  if (j0 + y < it.m && i0 + x < it.n) t[y][x] = it.r[(size_t)(j0 + y) * it.n + i0 + x];
  __syncthreads();
  if (i0 + y < it.n && j0 + x < it.m) {
    const double2 v = t[x][y];
    it.w[(size_t)(i0 + y) * it.m + j0 + x] = make_double2(v.x, -v.y);
  }
}

hipError_t launch_lq_adjoint(const LqItem* items_dev, int items, int max_rows, int max_len, hipStream_t s) {
  if (items <= 0 || max_rows <= 0 || max_len <= 0) return hipSuccess;
  const int tiles_m = cdiv(max_len, 16), per = cdiv(max_rows, 16) * tiles_m;
  hipLaunchKernelGGL(lq_adjoint_kernel, dim3(items * per), dim3(256), 0, s, items_dev, per, tiles_m);
  return hipGetLastError();
}

// sigma_i = ||a_i|| from the squared norms, stable descending order,
// k = min(cap, #{sigma > cutoff ||sigma||}) >= 1, lambda, scale and discarded
// weight as finalize_kernel; perm and 1 / sigma for the rows of V^+.
__global__ __launch_bounds__(1024) void lq_rank_kernel(const LqFinItem* items) {
  __shared__ double sig[1024];
  __shared__ int perm[1024];
  __shared__ int s_k;
  __shared__ double s_inv;
  const LqFinItem it = items[blockIdx.x];
  const int n = it.n, i = threadIdx.x;
  if (i < n) {
    sig[i] = sqrt(it.norm2[i]);
    perm[i] = i;
  }
  __syncthreads();
  if (i < n) {
    const double si = sig[i];
    int r = 0;
    for (int j = 0; j < n; ++j) {
      const double sj = sig[j];
      r += (sj > si) || (sj == si && j < i);
    }
    perm[r] = i;
  }
  __syncthreads();
  // sums over the ordered values: one wave, lane l takes l, l + 64, ...
  if (i < 64) {
    double tot = 0.0;
    for (int a = i; a < n; a += 64) tot += sig[a] * sig[a];
    tot = wave_sum(tot);
    const double nrm = sqrt(tot);
    int k = 0;
    for (int a = i; a < n; a += 64) k += sig[a] > it.cutoff * nrm ? 1 : 0;
    k = (int)wave_sum((double)k);
    k = min(max(k, 1), it.cap);
    double kept2 = 0.0, disc2 = 0.0;
    for (int a = i; a < n; a += 64) {
      const double sv = sig[perm[a]];
      if (a < k) kept2 += sv * sv;
      else disc2 += sv * sv;
    }
    kept2 = wave_sum(kept2);
    disc2 = wave_sum(disc2);
    const double kept = sqrt(kept2);
    const bool bad = !isfinite(tot) || !(kept > 0.0) || !isfinite(kept);
    if (i == 0) {
      *it.status_out = bad ? 1 : 0;
      s_inv = bad ? 0.0 : 1.0 / kept;
      *it.k_out = k;
      *it.scale_out = s_inv;
      *it.disc_out = tot > 0.0 ? disc2 / tot : 0.0;
      s_k = k;
    }
  }
  __syncthreads();
  if (i < s_k) {
    const double sv = sig[perm[i]];
    it.lam_out[i] = sv * s_inv;
    it.perm_out[i] = perm[i];
    it.inv_out[i] = sv > 0.0 ? 1.0 / sv : 0.0;
  }
}

hipError_t launch_lq_rank(const LqFinItem* items_dev, int items, hipStream_t s) {
  if (items <= 0) return hipSuccess;
  hipLaunchKernelGGL(lq_rank_kernel, dim3(items), dim3(1024), 0, s, items_dev);
  return hipGetLastError();
}

// V^+ (k x m) = Z Q1: row a of Z is the converged row perm[a] over its norm,
// row s of Q1 the s-th processed row of the first factorisation.
struct LqVecP {
  using T = double;
  using Ctx = LqVecItem;
  static constexpr bool A_CONTIG_K = true, B_CONTIG_N = true, REAL_ONLY = false;
  const LqVecItem* items;
  __device__ Ctx context(int i) const {
    LqVecItem t = items[i];
    t.k = min(t.k, *t.k_dev);
    return t;
  }
  __device__ static void dims(const Ctx& c, int& M, int& N, int& K) {
    M = c.k;
    N = c.m;
    K = c.n1;
  }
  struct RowA {
    const double2* z;
    double inv;
  };
  using ColB = const double2*;
  __device__ static RowA rowA(const Ctx& c, int i) {
    return RowA{c.z + (size_t)c.perm[i] * c.n1, c.inv[i]};
  }
  __device__ static ColB colB(const Ctx& c, int j) { return c.q + j; }
  __device__ static double2 loadA(const Ctx&, RowA r, int, int k) {
    const double2 v = r.z[k];
    return make_double2(v.x * r.inv, v.y * r.inv);
  }
  __device__ static double2 loadB(const Ctx& c, ColB b, int k, int) { return b[(size_t)c.order[k] * c.m]; }
  __device__ static void store(const Ctx& c, int i, int j, double re, double im) {
    c.v[(size_t)i * c.m + j] = make_double2(re, im);
  }
};

hipError_t launch_lq_vec(const LqVecItem* items_dev, int items, int max_k, int max_len, hipStream_t s) {
  LqVecP p{items_dev};
  return launch_cgemm<64, 64, 16>(p, items, max_k, max_len, s);
}

}  // namespace mps
