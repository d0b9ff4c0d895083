// Adaptive-lasso pruning of B0 / B_tau, the step after the fit that the paper names but does
// not specify.  Variable i (position k of the causal order) is regressed with intercept on its
// k predecessors at lag 0 and on all m variables at lags 1..p (d = k + m p columns).  The
// unpruned coefficients b are that regression's least-squares solution, so column j is scaled
// by |b_j| (adaptive lasso, Zou 2006, exponent 1).  The lasso path is the LARS path with the
// lasso modification (Efron, Hastie, Johnstone and Tibshirani 2004, Sec. 2 and Sec. 3.1), and
// the knot minimising BIC = T ln(RSS / T) + df ln T (df = nonzero coefficients) is kept.
//
// Everything the path needs is in one FP64 matrix: the centred cross-products C of the
// m (p + 1) lag-embedded columns, shared by all m regressions (lag 0 in the causal order, so a
// design's columns are two runs of consecutive columns of C).  One workgroup follows one
// variable's path on it.  Its state:
//   Li   the inverse of the Cholesky factor of the active columns' Gram (lower triangular,
//        G_A^{-1} = Li^T Li), in a region of global memory of its own.  A joining column appends
//        one row and leaves the others as they are; a leaving one rotates the rows below it;
//   q    G_A^{-1} s, bordered along with Li (recomputed from Li after a column leaves);
//   c    correlations z~_j^T r of the inactive columns with the current residual, updated by
//        c -= gamma a; an active column's is s_j C after every step (the equiangular property);
//   beta the scaled coefficients, best the coefficients of the best knot so far.
// The residual sum of squares follows from the step: the direction u has |u| = 1 and
// u^T r = C / A_A, so RSS falls by gamma (2 C / A_A - gamma).
// Numerical rules, shared with the FP64 reference: a step must exceed 1e-12 of the full step
// C / A_A; a column whose Schur complement against the active ones is <= 1e-12 of its squared
// norm is excluded; the path ends once C <= 1e-12 C_0, at the least-squares fit, or after the
// step limit (8 d by default).  Ties go to the lowest design column.
//
// What bounds it: memory.  A step with |A| of d columns active reads Li once (|A|^2 / 2
// doubles, private to the variable: 1.9 GB of them at m = 400, p = 2, far over the
// caches) and min(|A|, d - |A|) rows of C (shared, 11.5 MB: served by L2 and the Infinity Cache).
// Measured at m = 400, p = 2, n = 10^4, complete paths: 174 ms a call, 1.1 TB of both; 601 ms with the
// inverse of the active Gram itself kept and updated (1.25 |A|^2 doubles a step, written too).
// Clocks of the longest path (1199 columns): 74 ms in the products with C, 76 ms in those with
// Li, 9 ms in the rest; together the workgroups move ~9 TB/s through the caches.
#include "prune.hpp"
#include "gram.hpp"
#include "order_dev.hpp"
#include "profile.hpp"
#include "var_fit.hpp"


namespace vl {
namespace {

constexpr int kPT = 512;            // threads per variable
constexpr int kPW = kPT / kWave;
constexpr int kPanel = 1024;        // columns per pass when the state is in memory
constexpr int kMemNC = 20;          // pieces of an active set whose rows fit in registers there
constexpr int kMemMaxD = 4096;      // designs (m (p + 1) <= 4096)
constexpr double kGammaRel = 1e-12;
constexpr double kCollinearRel = 1e-12;
constexpr double kStopRel = 1e-12;
constexpr int kNone = 0x7fffffff;

struct PruneArgs {
  const double* C;
  int64_t ldc, m, T, cap;
  int p, dmax;
  const int32_t* order;
  const double* B0;
  const double* Bl;
  double* regions;
  double* B0o;
  double* Blo;
  int32_t* info;
  int32_t* st;
};

// Sum over the wave, the same bits in every lane (DPP and permlane butterflies).
__device__ inline double wave_allsum_d(double v) {
  v += dpp_f64<kDppRowMirror>(v);
  v += dpp_f64<kDppHalfMirror>(v);
  v += dpp_f64<kDppQuadXor2>(v);
  v += dpp_f64<kDppQuadXor1>(v);
  v += partner16_f64(v);
  v += partner32_f64(v);
  return v;
}

// Workgroup sums of two values, the same bits in every thread (waves in a fixed order).
__device__ inline void wg_sum2(double& a, double& b, double* red) {
  a = wave_allsum_d(a);
  b = wave_allsum_d(b);
  __syncthreads();
  if ((threadIdx.x & (kWave - 1)) == 0) {
    red[threadIdx.x / kWave] = a;
    red[kPW + threadIdx.x / kWave] = b;
  }
  __syncthreads();
  a = red[0];
  b = red[kPW];
#pragma unroll
  for (int w = 1; w < kPW; ++w) {
    a += red[w];
    b += red[kPW + w];
  }
}

__device__ inline double wg_sum(double v, double* red) {
  double z = 0.0;
  wg_sum2(v, z, red);
  return v;
}

// A candidate step: its length, the design column that breaks ties, the slot it is held in.
struct Cand {
  double g = INFINITY;
  int j = kNone, slot = kNone;
  __device__ inline void take(double g2, int j2, int s2) {
    if (g2 < g || (g2 == g && j2 < j)) {
      g = g2;
      j = j2;
      slot = s2;
    }
  }
};

// Smallest candidate of the wave, the lowest design column on ties, in every lane.
__device__ inline void wave_min_cand(Cand& x) {
  const double g = wave_min_quiet(x.g);
  const int j = wave_min_i32(x.g == g ? x.j : kNone);
  const int s = wave_min_i32(x.g == g && x.j == j ? x.slot : kNone);
  x.g = g;
  x.j = j;
  x.slot = s;
}

// Workgroup minima of two candidates, exact, so the same in every thread.
__device__ inline void wg_min2(Cand& x, Cand& y, double* rg, int* rj) {
  wave_min_cand(x);
  wave_min_cand(y);
  __syncthreads();
  if ((threadIdx.x & (kWave - 1)) == 0) {
    const int w = threadIdx.x / kWave;
    rg[w] = x.g;
    rg[kPW + w] = y.g;
    rj[w] = x.j;
    rj[kPW + w] = x.slot;
    rj[2 * kPW + w] = y.j;
    rj[3 * kPW + w] = y.slot;
  }
  __syncthreads();
  x = Cand{rg[0], rj[0], rj[kPW]};
  y = Cand{rg[kPW], rj[2 * kPW], rj[3 * kPW]};
#pragma unroll
  for (int w = 1; w < kPW; ++w) {
    x.take(rg[w], rj[w], rj[kPW + w]);
    y.take(rg[kPW + w], rj[2 * kPW + w], rj[3 * kPW + w]);
  }
}

// The lane index, opaque to the optimiser: what is derived from it is then formed where it is
// used.  Otherwise the row offsets below are hoisted out of the path's loop, held in registers
// across all of it, and spilled (129 registers at NC = 20).
__device__ __forceinline__ int fresh_lane() {
  int lane = threadIdx.x & (kWave - 1);
  asm volatile("" : "+v"(lane));
  return lane;
}

// Values every thread of the workgroup holds alike (read back from LDS after a reduction),
// declared uniform so they live in scalar registers and branch without divergence.
__device__ inline int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline int64_t uni64(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// ------------------------------------------------------------------------------------------
// Li, packed by blocks of 64 rows: block k holds rows 64 k .. 64 k + 63, each 64 (k + 1)
// doubles long (its entries, then zeros), so a wave reads a row as k + 1 aligned 512-byte
// pieces and the whole matrix is read in memory order.
// ------------------------------------------------------------------------------------------
__device__ inline int64_t li_row(int r) {
  const int64_t k = r >> 6;
  return 2048 * k * (k + 1) + (int64_t)(r & 63) * 64 * (k + 1);
}

// Rows of block k - 1 (k = K or K - 1 pieces a row) against x: the wave's rows 64 (k - 1) + w +
// 8 i, two at a time.  Each row stays in registers between its dot product y_r = Li_r x and its
// share of g += Li_r^T y_r, so Li is read once; ysq sums y_r^2.
template <int K, int NC>
__device__ __forceinline__ void li_block(const double* __restrict__ Li, int k, int n, int w,
                                         const double (&x)[NC], double (&g)[NC], double& ysq) {
  const double* B = Li + 2048 * (int64_t)(k - 1) * k + fresh_lane();
  const bool odd = k < K;
#pragma unroll 1
  for (int i = w; i < 64; i += 2 * kPW) {
    const int r = 64 * (k - 1) + i;
    if (r >= n) break;
    const bool two = r + kPW < n;
    const double* p0 = B + i * 64 * k;
    const double* p1 = two ? p0 + kPW * 64 * k : p0;
    double a0[K], a1[K];
#pragma unroll
    for (int c = 0; c < K - 1; ++c) a0[c] = p0[64 * c];
#pragma unroll
    for (int c = 0; c < K - 1; ++c) a1[c] = p1[64 * c];
    a0[K - 1] = a1[K - 1] = 0.0;
    if (!odd) {
      a0[K - 1] = p0[64 * (K - 1)];
      a1[K - 1] = p1[64 * (K - 1)];
    }
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int c = 0; c < K; ++c) {
      s0 = fma(a0[c], x[c], s0);
      s1 = fma(a1[c], x[c], s1);
    }
    s0 = wave_allsum_d(s0);
    s1 = two ? wave_allsum_d(s1) : 0.0;
    ysq = fma(s0, s0, ysq);
    ysq = fma(s1, s1, ysq);
#pragma unroll
    for (int c = 0; c < K; ++c) g[c] = fma(a1[c], s1, fma(a0[c], s0, g[c]));
  }
}

// Every block of rows; one instance per two piece counts keeps the loop's code (it runs through
// all of them each step) well inside the instruction cache.
template <int K, int NC>
__device__ __forceinline__ void li_blocks(const double* __restrict__ Li, int n, int w,
                                          const double (&x)[NC], double (&g)[NC], double& ysq) {
  const int nb = (n + 63) >> 6;
#pragma unroll 1
  for (int k = K - 1; k <= K && k <= nb; ++k) li_block<K, NC>(Li, k, n, w, x, g, ysq);
  if constexpr (K < NC) {
    if (K < nb) li_blocks<K + 2, NC>(Li, n, w, x, g, ysq);
  }
}

// The rest of apply_inverse's register form: g from the wave's rows, |Li x|^2, the waves' sums.
template <int NC>
__device__ __forceinline__ double apply_rows(const double* __restrict__ Li, int n, const double* x,
                                             double* out, double* part, double* red) {
  const int t = threadIdx.x, lane = fresh_lane(), w = uni(t / kWave);
  double ysq = 0.0, z = 0.0;
  double xr[NC], g[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    xr[c] = 64 * c < n ? x[64 * c + lane] : 0.0;
    g[c] = 0.0;
  }
  static_assert(NC % 2 == 0, "two piece counts an instance");
  li_blocks<2, NC>(Li, n, w, xr, g, ysq);
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int e = 64 * c + lane;
    if (e < n) part[w * n + e] = g[c];
  }
  ysq = lane == 0 ? ysq : 0.0;
  wg_sum2(ysq, z, red);
  for (int r = t; r < n; r += kPT) {
    double s = part[r];
#pragma unroll
    for (int q = 1; q < kPW; ++q) s += part[q * n + r];
    out[r] = s;
  }
  __syncthreads();
  return ysq;
}

// The same for any n <= kMemMaxD, Li read twice: y = Li x by rows, then Li^T y by panels of kPanel
// columns, a panel's sums in registers.  Both with two rows of 16 pieces in flight a wave; pieces
// past a row's end read its last one with weight 0.  part: kPW kPanel doubles (x in the first pass),
// y: kMemMaxD doubles, both LDS.
__device__ __forceinline__ double apply_passes(const double* __restrict__ Li, int n,
                                               const double* x, double* out, double* part,
                                               double* y, double* red) {
  constexpr int U = kPanel / kWave;
  const int t = threadIdx.x, lane = fresh_lane(), w = uni(t / kWave);
  double ysq = 0.0, z = 0.0;
  for (int e = t; e < 64 * ((n + 63) / 64); e += kPT) part[e] = x[e];
  __syncthreads();
#pragma unroll 1
  for (int r = w; r < n; r += 2 * kPW) {
    const bool two = r + kPW < n;
    const int r1 = two ? r + kPW : r, k0 = r >> 6, k1 = r1 >> 6;
    const double *p0 = Li + li_row(r) + lane, *p1 = Li + li_row(r1) + lane;
    double s0 = 0.0, s1 = 0.0;
#pragma unroll 1
    for (int c0 = 0; c0 <= k1; c0 += U) {
      double a0[U], a1[U];
#pragma unroll
      for (int u = 0; u < U; ++u) a0[u] = p0[64 * min(c0 + u, k0)];
#pragma unroll
      for (int u = 0; u < U; ++u) a1[u] = p1[64 * min(c0 + u, k1)];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const double xv = part[64 * min(c0 + u, k1) + lane];
        s0 = fma(a0[u], c0 + u <= k0 ? xv : 0.0, s0);
        s1 = fma(a1[u], c0 + u <= k1 ? xv : 0.0, s1);
      }
    }
    s0 = wave_allsum_d(s0);
    s1 = two ? wave_allsum_d(s1) : 0.0;
    ysq = fma(s0, s0, ysq);
    ysq = fma(s1, s1, ysq);
    if (lane == 0) {
      y[r] = s0;
      if (two) y[r1] = s1;
    }
  }
  ysq = lane == 0 ? ysq : 0.0;
  wg_sum2(ysq, z, red);                              // (its barriers: y is whole, x is done with)
#pragma unroll 1
  for (int e0 = 0; e0 < n; e0 += kPanel) {
    const int c0 = e0 >> 6;
    double g[U];
#pragma unroll
    for (int u = 0; u < U; ++u) g[u] = 0.0;
#pragma unroll 1
    for (int r = e0 + w; r < n; r += 2 * kPW) {
      const bool two = r + kPW < n;
      const int r1 = two ? r + kPW : r, k0 = r >> 6, k1 = r1 >> 6;
      const double *p0 = Li + li_row(r) + lane, *p1 = Li + li_row(r1) + lane;
      double a0[U], a1[U];
#pragma unroll
      for (int u = 0; u < U; ++u) a0[u] = p0[64 * min(c0 + u, k0)];
#pragma unroll
      for (int u = 0; u < U; ++u) a1[u] = p1[64 * min(c0 + u, k1)];
      const double y0 = y[r], y1 = two ? y[r1] : 0.0;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        g[u] = fma(a0[u], c0 + u <= k0 ? y0 : 0.0, g[u]);
        g[u] = fma(a1[u], c0 + u <= k1 ? y1 : 0.0, g[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) part[w * kPanel + 64 * u + lane] = g[u];
    __syncthreads();
    for (int e = t; e < min(kPanel, n - e0); e += kPT) {
      double s = part[e];
#pragma unroll
      for (int q = 1; q < kPW; ++q) s += part[q * kPanel + e];
      out[e0 + e] = s;
    }
    __syncthreads();
  }
  return ysq;
}

// out = G_A^{-1} x = Li^T (Li x) over n active slots; returns |Li x|^2 (every thread alike).  x
// holds zeros up to the next multiple of 64; x and out may not alias.  NC > 0: rows in registers,
// one read of Li (n <= 64 NC, x in LDS).  NC = 0: x in memory, the same while kMemNC pieces hold the
// active set, else two reads.  With this and the products by rows of C the complete paths at
// m = 400, p = 3 take 635 ms and at m = 660, p = 1 334 (16 pieces: 783 and 388; two reads with one
// load at a time: 2302 and 1416).  Ends with a barrier.
template <int NC>
__device__ __forceinline__ double apply_inverse(const double* __restrict__ Li, int n, const double* x,
                                                double* out, double* part, double* red) {
  if constexpr (NC > 0) {
    return apply_rows<NC>(Li, n, x, out, part, red);
  } else {
    if (n <= 64 * kMemNC) return apply_rows<kMemNC>(Li, n, x, out, part, red);
    return apply_passes(Li, n, x, out, part, part + 64 * kMemNC * kPW, red);
  }
}

// Removes active slot r0 of n from Li.  G_A^{-1} = sum of the rows' outer products; rotating row
// r0 into every row below it moves all of column r0 into that one row, whose outer product is
// then the Schur complement's term, and is dropped.  cs, sn, v, tmp: vectors of n.  Ends with a
// barrier.
__device__ __forceinline__ void li_remove(double* __restrict__ Li, int n, int r0, double* cs, double* sn,
                                 double* v, double* tmp) {
  const int t = threadIdx.x;
  // the rotations follow from column r0 alone
  for (int k = r0 + t; k < n; k += kPT) sn[k] = Li[li_row(k) + r0];
  for (int e = t; e < n; e += kPT) v[e] = e <= r0 ? Li[li_row(r0) + e] : 0.0;
  __syncthreads();
  if (t == 0) {
    double h = sn[r0];
    for (int k = r0 + 1; k < n; ++k) {
      const double b = sn[k], h2 = sqrt(fma(h, h, b * b));
      cs[k] = h / h2;
      sn[k] = b / h2;
      h = h2;
    }
  }
  __syncthreads();
  // row k against the carried row v, written to the place of row k - 1 with column r0 left out
  // once every thread has read its entries of both
  for (int k = r0 + 1; k < n; ++k) {
    const double* src = Li + li_row(k);
    double* dst = Li + li_row(k - 1);
    const double ck = cs[k], sk = sn[k];
    for (int e = t; e <= k; e += kPT) {
      const double b = src[e];
      tmp[e] = fma(ck, b, -sk * v[e]);
      v[e] = fma(sk, b, ck * v[e]);
    }
    __syncthreads();
    for (int e = t; e <= k; e += kPT)
      if (e != r0) dst[e < r0 ? e : e - 1] = tmp[e];
  }
  __syncthreads();
}

// permutation check of the order (one workgroup; m <= 4096)
__global__ __launch_bounds__(256) void prune_check_order_kernel(const int32_t* __restrict__ order,
                                                                int64_t m, int32_t* st) {
  __shared__ int seen[4096];
  for (int64_t e = threadIdx.x; e < m; e += 256) seen[e] = 0;
  __syncthreads();
  for (int64_t e = threadIdx.x; e < m; e += 256) {
    const int v = order[e];
    if (v < 0 || v >= m) raise_status(st, VL_ERR_INVALID_ARG);
    else atomicAdd(&seen[v], 1);
  }
  __syncthreads();
  for (int64_t e = threadIdx.x; e < m; e += 256)
    if (seen[e] != 1) raise_status(st, VL_ERR_INVALID_ARG);
}

// part[w np + e] = sum over the wave's eighth of the n active slots of C[col_r][ic_e] b_r, for
// np inactive columns ic: every wave has the same work whatever the split of active and inactive
// columns.  The slots' columns and weights go to scalar registers; 2 RU loads are in flight per
// lane (a row of C is read as coalesced pieces where the inactive columns are consecutive).
template <int RU>
__device__ __forceinline__ void inactive_dots(const double* __restrict__ C, int64_t ldc, int n,
                                     const int* col, const double* b, int np, const int* ic,
                                     double* part) {
  const int lane = fresh_lane(), w = uni(threadIdx.x / kWave);
  const int r0 = n * w / kPW, r1 = n * (w + 1) / kPW;
  for (int e0 = 0; e0 < np; e0 += 2 * kWave) {
    const int ea = e0 + lane, eb = ea + kWave;
    const int oa = ic[min(ea, np - 1)], ob = ic[min(eb, np - 1)];
    double sa[2] = {0.0, 0.0}, sb[2] = {0.0, 0.0};
    for (int rb = r0; rb < r1; rb += kWave) {
      const int rl = min(rb + lane, r1 - 1);
      const int cl = col[rl];
      const double bl = rb + lane < r1 ? b[rl] : 0.0;
      const int lo = __double2loint(bl), hi = __double2hiint(bl);
      const int nb = min(kWave, r1 - rb);
#pragma unroll 1
      for (int u0 = 0; u0 < nb; u0 += RU) {        // lanes past the end: weight 0
        double xa[RU], xb[RU];
#pragma unroll
        for (int u = 0; u < RU; ++u) {
          const double* row = C + (int64_t)__builtin_amdgcn_readlane(cl, u0 + u) * ldc;
          xa[u] = row[oa];
          xb[u] = row[ob];
        }
#pragma unroll
        for (int u = 0; u < RU; ++u) {
          const double wu = __hiloint2double(__builtin_amdgcn_readlane(hi, u0 + u),
                                             __builtin_amdgcn_readlane(lo, u0 + u));
          sa[u & 1] = fma(xa[u], wu, sa[u & 1]);
          sb[u & 1] = fma(xb[u], wu, sb[u & 1]);
        }
      }
    }
    if (ea < np) part[w * np + ea] = sa[0] + sa[1];
    if (eb < np) part[w * np + eb] = sb[0] + sb[1];
  }
}

// y[e] = sum_j C[ic_e][col_j] x_j over all d design columns (x: zero outside the active ones and up
// to the next multiple of 64) for np inactive columns ic; col_j = j, plus gap from pos on.  The
// other form of the same products, for more active columns than inactive ones.  A step then reads
// min(|A|, d - |A|) rows of C whole; by active rows alone the late steps read whole cache lines for
// a few scattered columns each (the longest path at m = 400, p = 2: 152 ms in these products by
// active rows alone, 71 ms with both forms).
// The columns 64 c0 .. 64 (c0 + K) - 1 of the design; kAdd: added to y (each entry by one lane).
template <int K, bool kAdd>
__device__ __forceinline__ void inactive_rows_k(const double* __restrict__ C, int64_t ldc, int d,
                                                int pos, int gap, const double* x, int np,
                                                const int* ic, double* y, int c0) {
  const int lane = fresh_lane(), w = uni(threadIdx.x / kWave);
  double xr[K];
  uint32_t k[K];
#pragma unroll
  for (int c = 0; c < K; ++c) {
    const int j = min(64 * (c0 + c) + lane, d - 1);
    k[c] = (uint32_t)(j + (j >= pos ? gap : 0));
    xr[c] = 64 * (c0 + c) < d ? x[64 * (c0 + c) + lane] : 0.0;
  }
#pragma unroll 1
  for (int e = w; e < np; e += 2 * kPW) {
    const bool two = e + kPW < np;
    const double* p0 = C + (int64_t)uni(ic[e]) * ldc;
    const double* p1 = C + (int64_t)uni(ic[two ? e + kPW : e]) * ldc;
    double a0[K], a1[K];
#pragma unroll
    for (int c = 0; c < K; ++c) a0[c] = p0[k[c]];
#pragma unroll
    for (int c = 0; c < K; ++c) a1[c] = p1[k[c]];
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int c = 0; c < K; ++c) {
      s0 = fma(a0[c], xr[c], s0);
      s1 = fma(a1[c], xr[c], s1);
    }
    s0 = wave_allsum_d(s0);
    s1 = wave_allsum_d(s1);
    if (lane == 0) {
      y[e] = kAdd ? y[e] + s0 : s0;
      if (two) y[e + kPW] = kAdd ? y[e + kPW] + s1 : s1;
    }
  }
}

// Any d: kMemNC pieces of the design at a time.
__device__ __forceinline__ void inactive_rows_any(const double* __restrict__ C, int64_t ldc, int d,
                                                  int pos, int gap, const double* x, int np,
                                                  const int* ic, double* y) {
  inactive_rows_k<kMemNC, false>(C, ldc, d, pos, gap, x, np, ic, y, 0);
#pragma unroll 1
  for (int c0 = kMemNC; 64 * c0 < d; c0 += kMemNC)
    inactive_rows_k<kMemNC, true>(C, ldc, d, pos, gap, x, np, ic, y, c0);
}

template <int K, int NC>
__device__ __forceinline__ void inactive_rows(const double* __restrict__ C, int64_t ldc, int d,
                                              int pos, int gap, const double* x, int np,
                                              const int* ic, double* y) {
  if (d <= 64 * K)
    inactive_rows_k<K, false>(C, ldc, d, pos, gap, x, np, ic, y, 0);
  else if constexpr (K < NC)
    inactive_rows<K + 2, NC>(C, ldc, d, pos, gap, x, np, ic, y);
}

// One workgroup per variable.  Active slots sit at the front of the state vectors, inactive
// columns (in design order until one leaves the active set) at their end, [ib, d).
//   NC > 0: the state vectors in LDS, designs of at most 64 NC columns;
//   NC = 0: any size, the state vectors in the region.
template <int NC>
__global__ __launch_bounds__(kPT) void prune_lars_kernel(PruneArgs a) {
  extern __shared__ double dyn[];
  __shared__ double red[2 * kPW], rg[2 * kPW];
  __shared__ int rj[4 * kPW], cnt[kPW];
  const int t = threadIdx.x, lane = t & (kWave - 1), wv = uni(t / kWave);
  const int64_t m = a.m, mp = m * a.p, ldc = a.ldc;
  const int64_t pos = m - 1 - (int64_t)blockIdx.x;  // the longest designs start first
  const int i = min(max(a.order[pos], 0), (int)m - 1);

  // this variable's region: after the regions of positions 0 .. pos-1
  double off = 0.0;
  for (int64_t k = t; k < pos; k += kPT) off += (double)prune_region_doubles(k + mp, a.cap);
  const int64_t base = uni64((int64_t)wg_sum(off, red));
  const int d = (int)(pos + mp);
  double* Li = a.regions + base;
  double* best = Li + prune_li_doubles(prune_active_cap(d, a.cap));
  // state vectors: scale; beta | correlation; q | Z~^T u; sign; two scratch vectors; column of C;
  // design column
  const int D = (int)round_up(NC > 0 ? a.dmax : d, 64);
  double* vec;
  if constexpr (NC > 0) vec = dyn;
  else vec = best + d;
  double* sc = vec;
  double* bc = sc + D;
  double* qa = bc + D;
  double* sv = qa + D;
  double* bv = sv + D;
  double* gn = bv + D;
  double *part, *more;                 // wave partials; scratch vectors of li_remove
  int* col;
  if constexpr (NC > 0) {
    part = gn + D;
    more = part;
    col = reinterpret_cast<int*>(part + kPW * D);
  } else {
    part = dyn;
    more = gn + D;
    col = reinterpret_cast<int*>(more + 4 * D);
  }
  int* des = col + D;
  const int panel = NC > 0 ? D : kPanel;

  // design columns: lag-0 predecessors in order, then (tau, k) for tau = 1..p, k = 0..m-1
  auto design = [&](int j, int& cj, double& s) {
    double bj;
    if (j < pos) {
      cj = j;
      bj = a.B0[(int64_t)i * m + min(max(a.order[j], 0), (int)m - 1)];
    } else {
      const int64_t jj = j - pos;
      cj = (int)(m + jj);
      bj = a.Bl[jj / m * m * m + (int64_t)i * m + jj % m];
    }
    s = fabs(bj);
  };
  double nkeep = 0.0, nok = 0.0;
  for (int j = t; j < d; j += kPT) {
    int cj;
    double s;
    design(j, cj, s);
    best[j] = 0.0;
    nkeep += s > 0.0 ? 1.0 : 0.0;
    nok += s > 0.0 && s * s * a.C[(int64_t)cj * ldc + cj] > 0.0 ? 1.0 : 0.0;
  }
  wg_sum2(nkeep, nok, red);
  int nA = 0, ib = d - uni((int)nok);
  Cand first, none;
  for (int j0 = 0, at = ib; j0 < d; j0 += kPT) {    // the usable columns, in design order
    const int j = j0 + t;
    int cj = 0;
    double s = 0.0;
    bool ok = false;
    if (j < d) {
      design(j, cj, s);
      ok = s > 0.0 && s * s * a.C[(int64_t)cj * ldc + cj] > 0.0;
    }
    const unsigned long long mk = __ballot(ok);
    if (lane == 0) cnt[wv] = __builtin_popcountll(mk);
    __syncthreads();
    int x = at + __builtin_popcountll(mk & ((1ull << lane) - 1ull));
#pragma unroll
    for (int w = 0; w < kPW; ++w) {
      x += w < wv ? cnt[w] : 0;
      at += cnt[w];
    }
    if (ok) {
      const double c = s * a.C[(int64_t)cj * ldc + pos];
      sc[x] = s;
      bc[x] = c;
      col[x] = cj;
      des[x] = j;
      first.take(-fabs(c), j, x);
    }
    __syncthreads();
  }
  wg_min2(first, none, rg, rj);
  const double C0 = first.j == kNone ? 0.0 : -first.g;
  const double T = (double)a.T, lnT = log(T);
  const double yy = a.C[pos * ldc + pos];
  double best_bic = T * log(yy / T), rss = yy, Cc = C0;
  int best_knot = 0, best_df = 0, steps = 0;
  const int64_t cap = a.cap > 0 ? a.cap : 8 * (int64_t)uni((int)nkeep);

  // inactive slot e leaves the list: the ones before it move up by one, kG groups of kPT at a time
  // (state in memory: their loads in flight together).  Every thread must be done with slot e before
  // the call; ends with a barrier.
  constexpr int kG = NC > 0 ? 1 : kMemMaxD / kPT;
  auto drop_inactive = [&](int e) {
    for (int hi = e - 1; hi >= ib; hi -= kG * kPT) {
      double v0[kG], v1[kG];
      int w0[kG], w1[kG];
#pragma unroll
      for (int q = 0; q < kG; ++q) {
        const int x = hi - t - q * kPT;
        v0[q] = v1[q] = 0.0;
        w0[q] = w1[q] = 0;
        if (x >= ib) {
          v0[q] = sc[x];
          v1[q] = bc[x];
          w0[q] = col[x];
          w1[q] = des[x];
        }
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < kG; ++q) {
        const int x = hi - t - q * kPT;
        if (x >= ib) {
          sc[x + 1] = v0[q];
          bc[x + 1] = v1[q];
          col[x + 1] = w0[q];
          des[x + 1] = w1[q];
        }
      }
    }
    ++ib;
    __syncthreads();
  };

  if (C0 > 0.0) {
    const int e = uni(first.slot), c1 = col[e], j1 = des[e];
    const double s1 = sc[e], sg = bc[e] >= 0.0 ? 1.0 : -1.0;
    const double g1 = s1 * s1 * a.C[(int64_t)c1 * ldc + c1];
    __syncthreads();
    drop_inactive(e);
    if (t < kWave) Li[t] = t == 0 ? 1.0 / sqrt(g1) : 0.0;
    if (t == 0) {
      sc[0] = s1;
      bc[0] = 0.0;
      qa[0] = sg / g1;
      sv[0] = sg;
      col[0] = c1;
      des[0] = j1;
    }
    nA = 1;
    __syncthreads();
  }

  while (nA > 0 && steps < cap) {
    // A_A = (s^T q)^(-1/2), direction A_A q
    double sq = 0.0;
    for (int r = t; r < nA; r += kPT) sq += sv[r] * qa[r];
    const double AA = 1.0 / sqrt(wg_sum(sq, red));
    for (int r = t; r < nA; r += kPT) bv[r] = sc[r] * (AA * qa[r]);
    __syncthreads();
    // a = Z~^T u for the inactive columns, the first of them to reach the active correlation
    // (gamma^), and the first active coefficient to change sign (gamma~)
    const double full = Cc / AA, tol = kGammaRel * full;
    Cand hat, til;
    const int nI = d - ib;
    for (int p0 = 0; p0 < nI; p0 += panel) {
      const int np = min(panel, nI - p0);
      if (p0 > 0) __syncthreads();
      const bool rows = nA > nI;
      if (rows) {
        if (p0 == 0) {
          for (int j = t; j < 64 * ((d + 63) / 64); j += kPT) gn[j] = 0.0;
          __syncthreads();
          for (int r = t; r < nA; r += kPT) gn[des[r]] = bv[r];
          __syncthreads();
        }
        if constexpr (NC > 0)
          inactive_rows<2, NC>(a.C, ldc, d, (int)pos, (int)(m - pos), gn, np, col + ib, part);
        else
          inactive_rows_any(a.C, ldc, d, (int)pos, (int)(m - pos), gn, np, col + ib + p0, part);
      } else {
        // up to four slots a wave: loads for four (m = 2040, p = 1, 25 steps: with drop_inactive's
        // loads in flight 19.0 -> 14.5 ms)
        if (NC == 0 && nA <= 4 * kPW)
          inactive_dots<4>(a.C, ldc, nA, col, bv, np, col + ib + p0, part);
        else
          inactive_dots<16>(a.C, ldc, nA, col, bv, np, col + ib + p0, part);
      }
      __syncthreads();
      for (int e = t; e < np; e += kPT) {
        double s = part[e];
        if (!rows) {
#pragma unroll
          for (int q = 1; q < kPW; ++q) s += part[q * np + e];
        }
        const int x = ib + p0 + e;
        const double aj = sc[x] * s, cj = bc[x];
        const int j = des[x];
        qa[x] = aj;
        double den = AA - aj;
        if (den != 0.0) {
          const double g = (Cc - cj) / den;
          if (isfinite(g) && g > tol) hat.take(g, j, x);
        }
        den = AA + aj;
        if (den != 0.0) {
          const double g = (Cc + cj) / den;
          if (isfinite(g) && g > tol) hat.take(g, j, x);
        }
      }
    }
    for (int r = t; r < nA; r += kPT) {
      const double dd = AA * qa[r];
      if (bc[r] != 0.0 && dd != 0.0) {
        const double g = -bc[r] / dd;
        if (g > tol) til.take(g, des[r], r);
      }
    }
    wg_min2(hat, til, rg, rj);
    const bool any = uni(hat.j) != kNone;
    const double gh = any ? hat.g : full;
    const int event = uni(til.g < gh ? -1 : any ? 1 : 0);
    const double gamma = event < 0 ? til.g : gh;
    const int r0 = event < 0 ? uni(til.slot) : -1;   // the leaving slot
    // move along the direction; df = nonzero coefficients of the columns that stay
    int nz = 0;
    for (int rb = 0; rb < nA; rb += kPT) {
      const int r = rb + t;
      bool on = false;
      if (r < nA) {
        const double b = bc[r] + gamma * (AA * qa[r]);
        bc[r] = b;
        on = b != 0.0 && r != r0;
      }
      nz += __builtin_popcountll(__ballot(on));
    }
    for (int x = ib + t; x < d; x += kPT) bc[x] -= gamma * qa[x];
    rss -= gamma * (2.0 * full - gamma);
    Cc -= gamma * AA;
    if (lane == 0) cnt[wv] = nz;
    __syncthreads();
    int df = 0;
#pragma unroll
    for (int w = 0; w < kPW; ++w) df += cnt[w];

    if (event < 0) {
      const double s0 = sc[r0], g0 = sv[r0] * Cc;
      const int c0 = col[r0], j0 = des[r0];
      __syncthreads();
      li_remove(Li, nA, r0, more, more + D, more + 2 * D, more + 3 * D);
      for (int lo = r0 + 1; lo < nA; lo += kPT) {
        const int x = lo + t;
        double v0 = 0.0, v1 = 0.0, v2 = 0.0;
        int w0 = 0, w1 = 0;
        if (x < nA) {
          v0 = sc[x];
          v1 = bc[x];
          v2 = sv[x];
          w0 = col[x];
          w1 = des[x];
        }
        __syncthreads();
        if (x < nA) {
          sc[x - 1] = v0;
          bc[x - 1] = v1;
          sv[x - 1] = v2;
          col[x - 1] = w0;
          des[x - 1] = w1;
        }
        __syncthreads();
      }
      --nA;
      --ib;
      if (t == 0) {
        sc[ib] = s0;
        bc[ib] = g0;
        col[ib] = c0;
        des[ib] = j0;
      }
      for (int r = t; r < 64 * ((nA + 63) / 64); r += kPT) bv[r] = r < nA ? sv[r] : 0.0;
      __syncthreads();
      apply_inverse<NC>(Li, nA, bv, qa, part, red);
    } else if (event > 0) {
      // border the factor with the joining column (or exclude it when collinear)
      const int e = uni(hat.slot), ck = col[e], jk = des[e];
      const double sk = sc[e], sgn = bc[e] >= 0.0 ? 1.0 : -1.0;
      const double* Ck = a.C + (int64_t)ck * ldc;     // C is symmetric
      const double gkk = sk * sk * Ck[ck];
      for (int r = t; r < 64 * ((nA + 63) / 64); r += kPT)
        bv[r] = r < nA ? sc[r] * sk * Ck[col[r]] : 0.0;
      __syncthreads();
      const double delta = gkk - apply_inverse<NC>(Li, nA, bv, gn, part, red);
      if (delta <= kCollinearRel * gkk) {
        drop_inactive(e);
      } else {
        // g = G_A^{-1} b: the new row of Li is [-g, 1] / sqrt(delta), and
        // q' = [q + g (g^T s - s_k) / delta, (s_k - g^T s) / delta]
        const double rd = 1.0 / delta, rs = 1.0 / sqrt(delta);
        double gp = 0.0;
        for (int x = t; x < nA; x += kPT) gp += gn[x] * sv[x];
        const double gs = wg_sum(gp, red);
        double* row = Li + li_row(nA);
        for (int x = t; x < 64 * (nA / 64 + 1); x += kPT)
          row[x] = x < nA ? -gn[x] * rs : (x == nA ? rs : 0.0);
        for (int x = t; x < nA; x += kPT) qa[x] += gn[x] * ((gs - sgn) * rd);
        drop_inactive(e);
        if (t == 0) {
          sc[nA] = sk;
          bc[nA] = 0.0;
          qa[nA] = (sgn - gs) * rd;
          sv[nA] = sgn;
          col[nA] = ck;
          des[nA] = jk;
        }
        ++nA;
        __syncthreads();
      }
    }
    ++steps;
    const double bic = T * log(rss / T) + (double)df * lnT;
    if (bic < best_bic) {
      best_bic = bic;
      best_knot = steps;
      best_df = df;
      // every column's entry: an excluded column is on neither list and may have been active at the
      // best knot before
      for (int j = t; j < d; j += kPT) best[j] = 0.0;
      __syncthreads();
      for (int r = t; r < nA; r += kPT) best[des[r]] = bc[r];
    }
    __syncthreads();
    if (event == 0 || Cc <= kStopRel * C0) break;
  }

  // outputs: row i of B0 (predecessors only) and of every B_tau.  They may be the inputs' own rows
  // (B0o = B0, Blo = Bl): every weight is read before the first output is written.
  for (int j = t; j < d; j += kPT) {
    int cj;
    double s;
    design(j, cj, s);
    best[j] *= s;
  }
  __syncthreads();
  double* rowB0 = a.B0o + (int64_t)i * m;
  for (int64_t v = t; v < m; v += kPT) rowB0[v] = 0.0;
  __syncthreads();
  for (int j = t; j < d; j += kPT) {
    if (j < pos) {
      rowB0[min(max(a.order[j], 0), (int)m - 1)] = best[j];
    } else {
      const int64_t jj = j - pos;
      a.Blo[jj / m * m * m + (int64_t)i * m + jj % m] = best[j];
    }
  }
  if (a.info && t == 0) {
    a.info[3 * i] = steps;
    a.info[3 * i + 1] = best_knot;
    a.info[3 * i + 2] = best_df;
  }
}

// LDS of the state vectors of a design of d columns: six FP64 vectors, the wave partials and two
// int32 vectors; the budget is a CU's 160 KiB
// less the kernel's static arrays.
constexpr size_t kPruneLds = 156 * 1024;
size_t prune_lds_bytes(int64_t d) {
  return (size_t)round_up(d, 64) * ((6 + kPW) * sizeof(double) + 2 * sizeof(int));
}

template <int NC>
int launch_prune(const PruneArgs& a, hipStream_t stream) {
  const size_t lds = NC > 0 ? prune_lds_bytes(a.dmax)
                            : (size_t)(kPW * 64 * kMemNC + kMemMaxD) * sizeof(double);
  static_assert(kPanel <= 64 * kMemNC, "the panels' partials fit in the rows'");
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(&prune_lars_kernel<NC>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
    return VL_ERR_HIP;
  prune_lars_kernel<NC><<<(unsigned)a.m, kPT, lds, stream>>>(a);
  VL_LAUNCH_CHECK();
  return VL_OK;
}

}  // namespace

size_t prune_ws_bytes(int64_t n, int64_t m, int p, int64_t cap, void* base, PruneWs* out) {
  Carver c(base);
  PruneWs w;
  const int64_t nc = m * (p + 1);
  w.colmap = c.take<int64_t>(nc);
  w.mu = c.take<double>(nc);
  w.C = c.take<double>(nc * nc);
  w.scratch = c.take<double>(lag_cov_scratch_doubles(n, m, p));
  int64_t tot = 0;
  for (int64_t k = 0; k < m; ++k) tot += prune_region_doubles(k + m * p, cap);
  w.regions = c.take<double>(tot);
  if (out) *out = w;
  return c.used;
}

int run_prune(int64_t n, int64_t m, int p, const PruneWs& w, const float* X, int64_t ldx,
              const int32_t* order, const double* B0, const double* Blag, int64_t cap,
              double* B0_out, double* Blag_out, int32_t* info, int32_t* st, hipStream_t stream) {
  ProfileScope ps("prune", stream);
  const int64_t nc = m * (p + 1);
  int rc = lag_covariance(n, m, p, X, ldx, order, w.colmap, w.mu, w.C, w.scratch, st, stream);
  if (rc) return rc;
  prune_check_order_kernel<<<1, 256, 0, stream>>>(order, m, st);
  VL_LAUNCH_CHECK();
  PruneArgs a;
  a.C = w.C;
  a.ldc = nc;
  a.m = m;
  a.T = n - p;
  a.cap = cap;
  a.p = p;
  a.order = order;
  a.B0 = B0;
  a.Bl = Blag;
  a.regions = w.regions;
  a.B0o = B0_out;
  a.Blo = Blag_out;
  a.info = info;
  a.st = st;
  // Rows of Li and C in registers and the state in LDS while both hold the longest design, by
  // register need; beyond that the general form.
  const int64_t d = m - 1 + m * p;
  a.dmax = (int)d;
  if (prune_lds_bytes(d) <= kPruneLds) {
    if (d <= 64 * 6) return launch_prune<6>(a, stream);
    if (d <= 64 * 10) return launch_prune<10>(a, stream);
    if (d <= 64 * 20) return launch_prune<20>(a, stream);
  }
  return launch_prune<0>(a, stream);
}

}  // namespace vl
