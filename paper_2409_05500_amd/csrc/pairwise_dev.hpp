// Device bodies of the pairwise-statistic precompute (Sec. 4.2 steps 1-2), shared by the
// single-problem kernels and the batched kernels.
#pragma once
#include <type_traits>

#include "common.hpp"

namespace vl {

// ------------------------------------------------------------------------------------------
// Stage 2a: standardise + transpose.  Block = 64 x 64 tile of E (t x i), staged through LDS.
// ------------------------------------------------------------------------------------------
__device__ inline void standardize_tile(
    const float* __restrict__ E, int64_t lde, int64_t n_eff, int64_t m,
    const double* __restrict__ mu, const double* __restrict__ cov, float* __restrict__ Xs,
    int64_t n_pad, int64_t m_pad, int32_t* st, int64_t t0, int64_t i0) {
  __shared__ float tile[64][65];
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const int64_t i = i0 + tx;
  double mui = 0.0, inv = 0.0;
  if (i < m) {
    const double var = cov[i * m + i];
    if (!(var > 0.0)) raise_status(st, VL_ERR_DEGENERATE);
    mui = mu[i];
    inv = var > 0.0 ? 1.0 / sqrt(var) : 0.0;
  }
  // every load of the tile in flight at once (a load under the bounds test would be waited for in
  // turn), by a stepped pointer clamped to the last row
  float ev[16];
  const float* Ei = E + (i < m ? i : m - 1);
  const float* last = Ei + (n_eff - 1) * lde;
  const float* pe = Ei + (t0 + ty) * lde;
#pragma unroll
  for (int q = 0; q < 16; ++q, pe += 4 * lde) ev[q] = *(pe < last ? pe : last);
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int r = ty + 4 * q;
    const float v = (float)(((double)ev[q] - mui) * inv);
    tile[r][tx] = i < m && t0 + r < n_eff ? v : 0.f;
  }
  __syncthreads();
  for (int r = ty; r < 64; r += 4) {
    const int64_t iv = i0 + r, t = t0 + tx;
    if (iv < m_pad && t < n_pad) Xs[iv * n_pad + t] = tile[tx][r];  // rows >= m get zeros
  }
}

// ------------------------------------------------------------------------------------------
// Stage 2b: moments of the standardised columns -> Hx.  One NT-thread block per variable; accurate
// library exp/log (O(mn) work, not on the critical path).
// ------------------------------------------------------------------------------------------
template <int NT>
__device__ __forceinline__ void hx_block(const float* __restrict__ Xs, int64_t n_pad, int64_t n_eff,
                                double* __restrict__ Hx, double* __restrict__ momx, int64_t i) {
  constexpr int kW = NT / 64;
  __shared__ double ra[kW], rb[kW];
  const float* x = Xs + i * n_pad;
  double sa = 0.0, sb = 0.0;
  auto term = [&](float u) {
    const float a = fabsf(u);
    sa += (double)(a + log1pf(expf(-2.f * a)) - (float)kLn2);
    sb += (double)(u * expf(-0.5f * u * u));
  };
  int64_t t = threadIdx.x;
  for (; t + 7 * NT < n_eff; t += 8 * NT) {  // eight loads in flight, summed in order
    float u[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) u[q] = x[t + q * NT];
#pragma unroll
    for (int q = 0; q < 8; ++q) term(u[q]);
  }
  if (t < n_eff) {                           // the last few, in flight together as well
    float u[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int64_t tq = t + q * NT;
      u[q] = x[tq < n_eff ? tq : n_eff - 1];
    }
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (t + q * NT < n_eff) term(u[q]);
  }
  sa = wave_sum_d(sa);
  sb = wave_sum_d(sb);
  if ((threadIdx.x & 63) == 0) {
    ra[threadIdx.x >> 6] = sa;
    rb[threadIdx.x >> 6] = sb;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double A = 0.0, B = 0.0;
#pragma unroll
    for (int w = 0; w < kW; ++w) {
      A += ra[w];
      B += rb[w];
    }
    A /= (double)n_eff;
    B /= (double)n_eff;
    Hx[i] = kHGauss - kK1 * (A - kGamma) * (A - kGamma) - kK2 * B * B;
    if (momx) {
      momx[2 * i] = A;
      momx[2 * i + 1] = B;
    }
  }
}

// ------------------------------------------------------------------------------------------
// Micro-tiles: kT x kT variable blocks {I, J} with bi <= bj, numbered row by row.
// ------------------------------------------------------------------------------------------
constexpr int kT = 4;

__device__ inline void tile_coords(int64_t k, int nt, int& bi, int& bj) {
  // upper-triangular tiles in row-major order: row r starts at r*nt - r*(r-1)/2
  const double T = (double)nt;
  const double disc = (2.0 * T + 1.0) * (2.0 * T + 1.0) - 8.0 * (double)k;
  int r = (int)(((2.0 * T + 1.0) - sqrt(disc > 0.0 ? disc : 0.0)) * 0.5);
  if (r < 0) r = 0;
  if (r > nt - 1) r = nt - 1;
  auto start = [nt](int q) { return (int64_t)q * nt - (int64_t)q * (q - 1) / 2; };
  while (r > 0 && start(r) > k) --r;
  while (r < nt - 1 && start(r + 1) <= k) ++r;
  bi = r;
  bj = r + (int)(k - start(r));
}

// A pair with sqrt(1 - rho^2) below kCollinearS is near-collinear: its Eq. 1 residual
// x_i - rho x_j cancels to a small fraction of the data, and forming it from the FP32 rounded
// standardised columns would amplify their rounding by 1 / sqrt(1 - rho^2).  The coefficient
// stage flags the micro-tiles that hold such a pair; their items are recomputed after the FP32
// moment kernel (which runs every tile), or taken instead of it where the items run as rows:
// standardised and with the residual formed in FP64 from E itself.
constexpr double kCollinearS = 0.25;

// One wave: from the flags clist[0 .. tiles) the number of flagged tiles, clist[tiles], and their
// list in tile order after it.
__device__ inline void list_collinear_tiles(int32_t* __restrict__ clist, int64_t tiles) {
  const int lane = threadIdx.x & 63;
  constexpr int kF = 16;                              // groups of 64 flags in flight
  int count = 0;
  for (int64_t t0 = 0; t0 < tiles; t0 += 64 * kF) {
    int32_t f[kF];
#pragma unroll
    for (int q = 0; q < kF; ++q) {
      const int64_t t = t0 + 64 * q + lane;
      f[q] = clist[t < tiles ? t : tiles - 1];
    }
#pragma unroll
    for (int q = 0; q < kF; ++q) {
      const int64_t t = t0 + 64 * q + lane;
      const bool on = t < tiles && f[q] != 0;
      const uint64_t hit = __ballot(on);
      if (on) clist[tiles + 1 + count + __builtin_popcountll(hit & ((1ull << lane) - 1ull))] = (int32_t)t;
      count += __builtin_popcountll(hit);
    }
  }
  if (lane == 0) clist[tiles] = count;
}

// ------------------------------------------------------------------------------------------
// Stage 3: scaled pair coefficients (a, b) of the micro-tiles {I, J}, bi <= bj (the others are
// read by nothing); zero on the diagonal / padding.  clist[tile] is 1 for a tile with a
// near-collinear pair, else 0.  One thread an entry, 16 consecutive threads a micro-tile: entry e
// of nt nt kT kT, so a tile's flag is one ballot and nothing has to be cleared first.
// ------------------------------------------------------------------------------------------
inline __host__ __device__ int64_t coef_threads(int64_t nt) { return nt * nt * kT * kT; }

__device__ inline void pair_coef_elem(const double* __restrict__ cov, int64_t m, int64_t m_pad,
                                      float2* __restrict__ coef, int nt,
                                      int32_t* __restrict__ clist, int32_t* st, int64_t e) {
  static_assert(kT * kT == 16, "a micro-tile is 16 lanes of a wave");
  const int64_t bi = (e >> 4) / nt, bj = (e >> 4) - bi * nt;
  const int64_t i = bi * kT + ((e >> 2) & 3), j = bj * kT + (e & 3);
  const bool own = bi <= bj && bi < nt;
  float2 c = make_float2(0.f, 0.f);
  bool near = false;
  if (own && i < m && j < m && i != j) {
    const double vi = cov[i * m + i], vj = cov[j * m + j];
    const double rho = cov[i * m + j] / sqrt(vi * vj);
    const double omr = 1.0 - rho * rho;
    near = !(omr >= kCollinearS * kCollinearS);
    if (!(omr >= kMinOneMinusRho2)) {
      raise_status(st, VL_ERR_DEGENERATE);
    } else {
      const double s = sqrt(omr);
      c = make_float2((float)(kWScale / s), (float)(kWScale * rho / s));
    }
  }
  const uint64_t any = __ballot(near);
  if (!own) return;
  coef[i * m_pad + j] = c;
  if ((e & 15) == 0)
    clist[bi * nt - bi * (bi - 1) / 2 + (bj - bi)] = (any >> (threadIdx.x & 48)) & 0xffff ? 1 : 0;
}

// ------------------------------------------------------------------------------------------
// Stage 4: the pairwise-moment kernel.
//
// Work item = (micro-tile of kT x kT variables {I, J} with bi <= bj, sample chunk).  One wave
// per item; lanes run over samples (2 consecutive samples per lane per step, float2 loads of
// the variable-major Xs; pairs outermost within a step), the kT*kT pair coefficients are
// wave-uniform (scalar registers).
// Per pair, sample and direction (w = c u):
//     q = w*w;  e = exp2(-q)  (= exp(-u^2/2));        Bacc += w * e
//     t = exp2(kTScale * |w|) (= exp(-2|u|));         P    *= (1 + t)
//     Uacc += |w|
// log cosh u = |u| + ln(1 + exp(-2|u|)) - ln 2, so the logarithm is taken once per 64
// samples of a lane from the running product P (each factor lies in (1, 2], P <= 2^64):
//     Uacc += c ln2 (log2 P - count),  P = 1
// which leaves Uacc = c * sum log cosh u exactly in real arithmetic.  Zero-padded samples
// give w = 0, t = 1, factor 2: they add exactly 0 to Uacc and Bacc.
// Two transcendentals and seven other VALU operations per (pair, sample, direction); the
// compensated variant adds three per sum (Kahan), 13 in all.
//
// At the end the 2 x 2 x kT x kT wave sums are formed by a reduce-scatter (lane l ends with
// value l) and written to per-chunk FP32 partials part{U,B}[chunk][row][col].
// ------------------------------------------------------------------------------------------
static_assert(2 * 2 * kT * kT == 64, "reduce-scatter expects 64 values per lane");

__device__ __forceinline__ void moment_step(float w, float& U, float& P, float& B) {
  const float q = w * w;
  const float e = __builtin_amdgcn_exp2f(-q);
  B = fmaf(w, e, B);
  const float aw = fabsf(w);
  const float t = __builtin_amdgcn_exp2f(aw * (float)kTScale);
  P = fmaf(P, t, P);
  U += aw;
}

// Kahan accumulation s += x: the true sum is s - c.
__device__ __forceinline__ void kahan_add(float& s, float& c, float x) {
  const float y = x - c;
  const float t = s + y;
  c = (t - s) - y;
  s = t;
}

// The moment accumulators of one (pair, direction), fed w = c u sample by sample: U sums |w|
// (and at each flush the log term of the running product P), B sums w e.  Plain FP32 sums
// (Comp = false), or Kahan-compensated ones (Comp = true): the compensation terms cU, cB keep
// a lane's sums within a few units of their last place whatever the sample count, where a
// plain running sum's rounding grows with it.
template <bool Comp>
struct MomentAcc;

template <>
struct MomentAcc<false> {
  float U, P, B;
  __device__ __forceinline__ void init() {
    U = 0.f;
    P = 1.f;
    B = 0.f;
  }
  __device__ __forceinline__ void step(float w) {
    const float q = w * w;
    const float e = __builtin_amdgcn_exp2f(-q);
    B = fmaf(w, e, B);
    const float aw = fabsf(w);
    const float t = __builtin_amdgcn_exp2f(aw * (float)kTScale);
    P = fmaf(P, t, P);
    U += aw;
  }
  __device__ __forceinline__ void flush(float cnt, float cln2) {
    U = fmaf(__builtin_amdgcn_logf(P) - cnt, cln2, U);
    P = 1.f;
  }
  __device__ __forceinline__ float u() const { return U; }
  __device__ __forceinline__ float b() const { return B; }
};

template <>
struct MomentAcc<true> {
  float U, cU, P, B, cB;
  __device__ __forceinline__ void init() {
    U = cU = B = cB = 0.f;
    P = 1.f;
  }
  __device__ __forceinline__ void step(float w) {
    const float q = w * w;
    const float e = __builtin_amdgcn_exp2f(-q);
    const float yb = fmaf(w, e, -cB);      // the product enters with one rounding
    const float tb = B + yb;
    cB = (tb - B) - yb;
    B = tb;
    const float aw = fabsf(w);
    const float t = __builtin_amdgcn_exp2f(aw * (float)kTScale);
    P = fmaf(P, t, P);
    kahan_add(U, cU, aw);
  }
  __device__ __forceinline__ void flush(float cnt, float cln2) {
    const float y = fmaf(__builtin_amdgcn_logf(P) - cnt, cln2, -cU);
    const float t = U + y;
    cU = (t - U) - y;
    U = t;
    P = 1.f;
  }
  __device__ __forceinline__ double u() const { return (double)U - (double)cU; }
  __device__ __forceinline__ double b() const { return (double)B - (double)cB; }
};

// Writes the 2 x 2 x kT x kT wave sums of one item: a reduce-scatter (lane l ends with value
// l), then the chunk partials part{U,B}[chunk][row][col] of the valid ordered pairs.  FP32
// partials take the plain sums (FP32 reduce-scatter); FP64 partials the compensated ones
// (each lane's exact value U - cU in FP64, FP64 reduce-scatter).
template <class TP, bool Comp>
__device__ __forceinline__ void write_moment_partials(MomentAcc<Comp> (&acc)[2][kT][kT],
                                                      int64_t i0, int64_t j0, int64_t m,
                                                      int64_t chunk, TP* __restrict__ partU,
                                                      TP* __restrict__ partB) {
  static_assert(std::is_same<TP, double>::value == Comp, "FP64 partials with compensation");
  const int lane = threadIdx.x & 63;
  // value index v = kind*32 + d*16 + ii*4 + jj (kind 0: U, 1: B)
  TP v[64];
#pragma unroll
  for (int d = 0; d < 2; ++d)
#pragma unroll
    for (int ii = 0; ii < kT; ++ii)
#pragma unroll
      for (int jj = 0; jj < kT; ++jj) {
        v[d * 16 + ii * 4 + jj] = acc[d][ii][jj].u();
        v[32 + d * 16 + ii * 4 + jj] = acc[d][ii][jj].b();
      }
  TP sum;
  if constexpr (Comp)
    sum = wave_reduce_scatter64_d(v);
  else
    sum = wave_reduce_scatter64(v);
  const int kind = lane >> 5, d = (lane >> 4) & 1, ii = (lane >> 2) & 3, jj = lane & 3;
  const int64_t i = i0 + ii, j = j0 + jj;
  if (i < m && j < m && i != j) {
    const int64_t row = d ? j : i, col = d ? i : j;
    TP* dst = kind ? partB : partU;
    dst[chunk * m * m + row * m + col] = sum;
  }
}

// One wave's work item (tile, chunk); item < items is the caller's check.  Always inlined:
// as a call its register use rises from 168 to 248 and the occupancy falls to 2 waves/SIMD.
__device__ __attribute__((always_inline)) inline void pairwise_moments_item(
    const float* __restrict__ Xs, int64_t n_pad, const float2* __restrict__ coef, int64_t m_pad,
    int64_t m, int nt, int64_t tiles, int chunk_len, int64_t item,
    float* __restrict__ partU, float* __restrict__ partB) {
  const int lane = threadIdx.x & 63;
  const int64_t chunk = item / tiles;
  const int64_t tile = item - chunk * tiles;
  int bi, bj;
  tile_coords(tile, nt, bi, bj);
  const int64_t i0 = (int64_t)bi * kT, j0 = (int64_t)bj * kT;

  float ca[kT][kT], cb[kT][kT];
#pragma unroll
  for (int ii = 0; ii < kT; ++ii)
#pragma unroll
    for (int jj = 0; jj < kT; ++jj) {
      // read-only for this kernel: the constant address space lets these wave-uniform loads
      // be scalar loads into SGPRs whatever the pointer's provenance
      typedef const __attribute__((address_space(4))) float* const_f32p;
      const const_f32p cp = (const_f32p)(uintptr_t)coef;
      const int64_t ci = 2 * ((i0 + ii) * m_pad + j0 + jj);
      const float2 c = make_float2(cp[ci], cp[ci + 1]);
      ca[ii][jj] = c.x;
      cb[ii][jj] = c.y;
    }

  float U[2][kT][kT], P[2][kT][kT], B[2][kT][kT];
#pragma unroll
  for (int d = 0; d < 2; ++d)
#pragma unroll
    for (int ii = 0; ii < kT; ++ii)
#pragma unroll
      for (int jj = 0; jj < kT; ++jj) {
        U[d][ii][jj] = 0.f;
        P[d][ii][jj] = 1.f;
        B[d][ii][jj] = 0.f;
      }

  // uniform row bases (scalar registers) and one 32-bit per-lane sample offset; 2 consecutive
  // samples per lane per step keep the live state at 168 VGPRs (3 waves per SIMD)
  const uint32_t tb = (uint32_t)(chunk * chunk_len) + 2u * (uint32_t)lane;
  const float* xi_r[kT];
  const float* xj_r[kT];
#pragma unroll
  for (int k = 0; k < kT; ++k) {
    xi_r[k] = Xs + (i0 + k) * n_pad;
    xj_r[k] = Xs + (j0 + k) * n_pad;
  }
  const float cln2 = (float)(kWScale * kLn2);
  const int steps = chunk_len / 128;                // 2 samples per lane per step
  int since_flush = 0;
  for (int s = 0; s < steps; ++s) {
    float2 xi[kT], xj[kT];
#pragma unroll
    for (int k = 0; k < kT; ++k) {
      const uint32_t o = tb + 128u * (uint32_t)s;
      xi[k] = *reinterpret_cast<const float2*>(xi_r[k] + o);
      xj[k] = *reinterpret_cast<const float2*>(xj_r[k] + o);
    }
#pragma unroll
    for (int ii = 0; ii < kT; ++ii) {
#pragma unroll
      for (int jj = 0; jj < kT; ++jj) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const float xv = e ? xi[ii].y : xi[ii].x;
          const float yv = e ? xj[jj].y : xj[jj].x;
          const float w0 = fmaf(xv, ca[ii][jj], -(yv * cb[ii][jj]));
          const float w1 = fmaf(yv, ca[ii][jj], -(xv * cb[ii][jj]));
          moment_step(w0, U[0][ii][jj], P[0][ii][jj], B[0][ii][jj]);
          moment_step(w1, U[1][ii][jj], P[1][ii][jj], B[1][ii][jj]);
        }
      }
    }
    since_flush += 2;
    if (since_flush == 64 || s == steps - 1) {
      const float cnt = (float)since_flush;
#pragma unroll
      for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int ii = 0; ii < kT; ++ii)
#pragma unroll
          for (int jj = 0; jj < kT; ++jj) {
            U[d][ii][jj] = fmaf(__builtin_amdgcn_logf(P[d][ii][jj]) - cnt, cln2, U[d][ii][jj]);
            P[d][ii][jj] = 1.f;
          }
      since_flush = 0;
    }
  }

  // value index v = kind*32 + d*16 + ii*4 + jj (kind 0: U, 1: B)
  float v[64];
#pragma unroll
  for (int d = 0; d < 2; ++d)
#pragma unroll
    for (int ii = 0; ii < kT; ++ii)
#pragma unroll
      for (int jj = 0; jj < kT; ++jj) {
        v[d * 16 + ii * 4 + jj] = U[d][ii][jj];
        v[32 + d * 16 + ii * 4 + jj] = B[d][ii][jj];
      }
  const float sum = wave_reduce_scatter64(v);
  const int kind = lane >> 5, d = (lane >> 4) & 1, ii = (lane >> 2) & 3, jj = lane & 3;
  const int64_t i = i0 + ii, j = j0 + jj;
  if (i < m && j < m && i != j) {
    const int64_t row = d ? j : i, col = d ? i : j;
    float* dst = kind ? partB : partU;
    dst[chunk * m * m + row * m + col] = sum;
  }
}

// One row of a work item: variable i0 + row against the tile's kT columns, both directions.  The
// samples of a lane, the order of its sums, the flushes and the lane pairing of the reduction are
// the whole item's, so the partials are the same bits; a plan with few items then has four times
// the waves, each a quarter as long.
__device__ __attribute__((always_inline)) inline void pairwise_moments_row(
    const float* __restrict__ Xs, int64_t n_pad, const float2* __restrict__ coef, int64_t m_pad,
    int64_t m, int nt, int64_t tiles, int chunk_len, int64_t item, int row,
    float* __restrict__ partU, float* __restrict__ partB) {
  const int lane = threadIdx.x & 63;
  const int64_t chunk = item / tiles;
  const int64_t tile = item - chunk * tiles;
  int bi, bj;
  tile_coords(tile, nt, bi, bj);
  const int64_t i = (int64_t)bi * kT + row, j0 = (int64_t)bj * kT;
  if (i >= m) return;
  float ca[kT], cb[kT];
#pragma unroll
  for (int jj = 0; jj < kT; ++jj) {
    typedef const __attribute__((address_space(4))) float* const_f32p;
    const const_f32p cp = (const_f32p)(uintptr_t)coef;
    const int64_t ci = 2 * (i * m_pad + j0 + jj);
    ca[jj] = cp[ci];
    cb[jj] = cp[ci + 1];
  }
  float U[2][kT], P[2][kT], B[2][kT];
#pragma unroll
  for (int d = 0; d < 2; ++d)
#pragma unroll
    for (int jj = 0; jj < kT; ++jj) {
      U[d][jj] = 0.f;
      P[d][jj] = 1.f;
      B[d][jj] = 0.f;
    }
  const uint32_t tb = (uint32_t)(chunk * chunk_len) + 2u * (uint32_t)lane;
  const float* xi_r = Xs + i * n_pad;
  const float* xj_r[kT];
#pragma unroll
  for (int k = 0; k < kT; ++k) xj_r[k] = Xs + (j0 + k) * n_pad;
  const float cln2 = (float)(kWScale * kLn2);
  const int steps = chunk_len / 128;
  int since_flush = 0;
  for (int s = 0; s < steps; ++s) {
    const uint32_t o = tb + 128u * (uint32_t)s;
    const float2 xi = *reinterpret_cast<const float2*>(xi_r + o);
    float2 xj[kT];
#pragma unroll
    for (int k = 0; k < kT; ++k) xj[k] = *reinterpret_cast<const float2*>(xj_r[k] + o);
#pragma unroll
    for (int jj = 0; jj < kT; ++jj) {
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const float xv = e ? xi.y : xi.x;
        const float yv = e ? xj[jj].y : xj[jj].x;
        const float w0 = fmaf(xv, ca[jj], -(yv * cb[jj]));
        const float w1 = fmaf(yv, ca[jj], -(xv * cb[jj]));
        moment_step(w0, U[0][jj], P[0][jj], B[0][jj]);
        moment_step(w1, U[1][jj], P[1][jj], B[1][jj]);
      }
    }
    since_flush += 2;
    if (since_flush == 64 || s == steps - 1) {
      const float cnt = (float)since_flush;
#pragma unroll
      for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int jj = 0; jj < kT; ++jj) {
          U[d][jj] = fmaf(__builtin_amdgcn_logf(P[d][jj]) - cnt, cln2, U[d][jj]);
          P[d][jj] = 1.f;
        }
      since_flush = 0;
    }
  }
  // value index v = kind*8 + d*4 + jj; lanes 4 v .. 4 v + 3 hold its sum
  float v[16];
#pragma unroll
  for (int d = 0; d < 2; ++d)
#pragma unroll
    for (int jj = 0; jj < kT; ++jj) {
      v[d * 4 + jj] = U[d][jj];
      v[8 + d * 4 + jj] = B[d][jj];
    }
  const float sum = wave_reduce_scatter16(v);
  const int kind = lane >> 5, d = (lane >> 4) & 1, jj = (lane >> 2) & 3;
  const int64_t j = j0 + jj;
  if ((lane & 3) == 0 && j < m && i != j) {
    const int64_t r = d ? j : i, c = d ? i : j;
    float* dst = kind ? partB : partU;
    dst[chunk * m * m + r * m + c] = sum;
  }
}

// The same work item with Kahan-compensated sums and FP64 partials (231 VGPRs, 2 waves per
// SIMD).  A separate body: folding both forms into one template changed the schedule the
// compiler chose for the plain one (6% slower).
__device__ __attribute__((always_inline)) inline void pairwise_moments_item_comp(
    const float* __restrict__ Xs, int64_t n_pad, const float2* __restrict__ coef, int64_t m_pad,
    int64_t m, int nt, int64_t tiles, int chunk_len, int64_t item,
    double* __restrict__ partU, double* __restrict__ partB) {
  constexpr bool Comp = true;
  const int lane = threadIdx.x & 63;
  const int64_t chunk = item / tiles;
  const int64_t tile = item - chunk * tiles;
  int bi, bj;
  tile_coords(tile, nt, bi, bj);
  const int64_t i0 = (int64_t)bi * kT, j0 = (int64_t)bj * kT;

  float ca[kT][kT], cb[kT][kT];
#pragma unroll
  for (int ii = 0; ii < kT; ++ii)
#pragma unroll
    for (int jj = 0; jj < kT; ++jj) {
      // read-only for this kernel: the constant address space lets these wave-uniform loads
      // be scalar loads into SGPRs whatever the pointer's provenance
      typedef const __attribute__((address_space(4))) float* const_f32p;
      const const_f32p cp = (const_f32p)(uintptr_t)coef;
      const int64_t ci = 2 * ((i0 + ii) * m_pad + j0 + jj);
      const float2 c = make_float2(cp[ci], cp[ci + 1]);
      ca[ii][jj] = c.x;
      cb[ii][jj] = c.y;
    }

  MomentAcc<Comp> acc[2][kT][kT];
#pragma unroll
  for (int d = 0; d < 2; ++d)
#pragma unroll
    for (int ii = 0; ii < kT; ++ii)
#pragma unroll
      for (int jj = 0; jj < kT; ++jj) acc[d][ii][jj].init();

  // uniform row bases (scalar registers) and one 32-bit per-lane sample offset; 2 consecutive
  // samples per lane per step keep the live state at 168 VGPRs (3 waves per SIMD)
  const uint32_t tb = (uint32_t)(chunk * chunk_len) + 2u * (uint32_t)lane;
  const float* xi_r[kT];
  const float* xj_r[kT];
#pragma unroll
  for (int k = 0; k < kT; ++k) {
    xi_r[k] = Xs + (i0 + k) * n_pad;
    xj_r[k] = Xs + (j0 + k) * n_pad;
  }
  const float cln2 = (float)(kWScale * kLn2);
  const int steps = chunk_len / 128;                // 2 samples per lane per step
  int since_flush = 0;
  for (int s = 0; s < steps; ++s) {
    float2 xi[kT], xj[kT];
#pragma unroll
    for (int k = 0; k < kT; ++k) {
      const uint32_t o = tb + 128u * (uint32_t)s;
      xi[k] = *reinterpret_cast<const float2*>(xi_r[k] + o);
      xj[k] = *reinterpret_cast<const float2*>(xj_r[k] + o);
    }
#pragma unroll
    for (int ii = 0; ii < kT; ++ii) {
#pragma unroll
      for (int jj = 0; jj < kT; ++jj) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const float xv = e ? xi[ii].y : xi[ii].x;
          const float yv = e ? xj[jj].y : xj[jj].x;
          const float w0 = fmaf(xv, ca[ii][jj], -(yv * cb[ii][jj]));
          const float w1 = fmaf(yv, ca[ii][jj], -(xv * cb[ii][jj]));
          acc[0][ii][jj].step(w0);
          acc[1][ii][jj].step(w1);
        }
      }
    }
    since_flush += 2;
    if (since_flush == 64 || s == steps - 1) {
      const float cnt = (float)since_flush;
#pragma unroll
      for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int ii = 0; ii < kT; ++ii)
#pragma unroll
          for (int jj = 0; jj < kT; ++jj) acc[d][ii][jj].flush(cnt, cln2);
      since_flush = 0;
    }
  }
  (void)lane;
  write_moment_partials(acc, i0, j0, m, chunk, partU, partB);
}

// The same item, (tile, chunk), for a flagged micro-tile.  Lanes run over samples, one per step.
// Each sample of the tile's 2 kT variables is standardised in FP64 from E (x = (e - mu) / sd, population moments), the residuals of
// both directions are formed in FP64, d = x_i - rho x_j, and only the scaled residual
// w = d c / sqrt(1 - rho^2) is rounded to FP32: its relative error is then that of one
// rounding, as for a well-conditioned pair.  The moment terms are the fast item's.
template <class TP>
__device__ __forceinline__ void pairwise_collinear_item(
    const float* __restrict__ E, int64_t lde, int64_t n_eff, const double* __restrict__ mu,
    const double* __restrict__ cov, int64_t m, int nt, int chunk_len, int64_t tile,
    int64_t chunk, TP* __restrict__ partU, TP* __restrict__ partB) {
  constexpr bool Comp = std::is_same<TP, double>::value;
  const int lane = threadIdx.x & 63;
  int bi, bj;
  tile_coords(tile, nt, bi, bj);
  const int64_t i0 = (int64_t)bi * kT, j0 = (int64_t)bj * kT;
  double mi[kT], si[kT], mj[kT], sj[kT];
  int64_t ci[kT], cj[kT];
#pragma unroll
  for (int k = 0; k < kT; ++k) {
    const bool oi = i0 + k < m, oj = j0 + k < m;
    ci[k] = oi ? i0 + k : m - 1;
    cj[k] = oj ? j0 + k : m - 1;
    mi[k] = mu[ci[k]];
    mj[k] = mu[cj[k]];
    si[k] = oi ? 1.0 / sqrt(cov[ci[k] * m + ci[k]]) : 0.0;   // padding variables: x = 0
    sj[k] = oj ? 1.0 / sqrt(cov[cj[k] * m + cj[k]]) : 0.0;
  }
  double rho[kT][kT], kc[kT][kT];
#pragma unroll
  for (int ii = 0; ii < kT; ++ii)
#pragma unroll
    for (int jj = 0; jj < kT; ++jj) {
      const int64_t i = i0 + ii, j = j0 + jj;
      rho[ii][jj] = 0.0;
      kc[ii][jj] = 0.0;
      if (i < m && j < m && i != j) {
        const double r = cov[i * m + j] / sqrt(cov[i * m + i] * cov[j * m + j]);
        const double omr = 1.0 - r * r;
        rho[ii][jj] = r;
        kc[ii][jj] = omr >= kMinOneMinusRho2 ? kWScale / sqrt(omr) : 0.0;  // else: raised
      }
    }

  MomentAcc<Comp> acc[2][kT][kT];
#pragma unroll
  for (int d = 0; d < 2; ++d)
#pragma unroll
    for (int ii = 0; ii < kT; ++ii)
#pragma unroll
      for (int jj = 0; jj < kT; ++jj) acc[d][ii][jj].init();
  const float cln2 = (float)(kWScale * kLn2);
  const int steps = chunk_len / 64;
  int since_flush = 0;
  for (int s = 0; s < steps; ++s) {
    const int64_t t = chunk * chunk_len + (int64_t)s * 64 + lane;
    const bool ot = t < n_eff;
    const int64_t tc = ot ? t : n_eff - 1;           // clamped row; padding samples give 0
    double xi[kT], xj[kT];
#pragma unroll
    for (int k = 0; k < kT; ++k) {
      xi[k] = mask_f64(((double)E[tc * lde + ci[k]] - mi[k]) * si[k], ot);
      xj[k] = mask_f64(((double)E[tc * lde + cj[k]] - mj[k]) * sj[k], ot);
    }
#pragma unroll
    for (int ii = 0; ii < kT; ++ii)
#pragma unroll
      for (int jj = 0; jj < kT; ++jj) {
        const float w0 = (float)(fma(-rho[ii][jj], xj[jj], xi[ii]) * kc[ii][jj]);
        const float w1 = (float)(fma(-rho[ii][jj], xi[ii], xj[jj]) * kc[ii][jj]);
        acc[0][ii][jj].step(w0);
        acc[1][ii][jj].step(w1);
      }
    since_flush += 1;
    if (since_flush == 64 || s == steps - 1) {
      const float cnt = (float)since_flush;
#pragma unroll
      for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int ii = 0; ii < kT; ++ii)
#pragma unroll
          for (int jj = 0; jj < kT; ++jj) acc[d][ii][jj].flush(cnt, cln2);
      since_flush = 0;
    }
  }
  write_moment_partials(acc, i0, j0, m, chunk, partU, partB);
}

// ------------------------------------------------------------------------------------------
// Stage 5: FP64 combine.  Hr[i][j] from the chunk partials (fixed order), then S.
// ------------------------------------------------------------------------------------------
__device__ inline double combine_finish(double su, double sb, int64_t n_eff, double* mom) {
  const double A = su / (kWScale * (double)n_eff);
  const double B = sb / (kWScale * (double)n_eff);
  if (mom) {
    mom[0] = A;
    mom[1] = B;
  }
  return kHGauss - kK1 * (A - kGamma) * (A - kGamma) - kK2 * B * B;
}

// Block bi <= bj of kCS x kCS entries and its mirror image, one entry of each a thread: Hr of both
// (partials read along rows, four chunks of both in flight, added in chunk order), then S of
// both, the mirrored Hr passing through LDS: the same two sums in both orders -> S[j][i] ==
// -S[i][j] bit for bit.  kCS^2 threads.
constexpr int kCS = 16;

template <class TP>
__device__ __forceinline__ void combine_score_block(const TP* __restrict__ partU,
                                           const TP* __restrict__ partB, int nc, int64_t m,
                                           int64_t n_eff, const double* __restrict__ Hx,
                                           double* __restrict__ Hr, double* __restrict__ mom,
                                           double* __restrict__ S, int64_t bi, int64_t bj) {
  __shared__ double h[2][kCS][kCS + 1];
  const int tx = threadIdx.x % kCS, ty = threadIdx.x / kCS;
  int64_t i[2], j[2], e[2];
  bool in[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    i[q] = (q ? bj : bi) * kCS + ty;
    j[q] = (q ? bi : bj) * kCS + tx;
    in[q] = i[q] < m && j[q] < m;
    e[q] = in[q] ? i[q] * m + j[q] : 0;
  }
  const int64_t mm = m * m;
  double su[2] = {0.0, 0.0}, sb[2] = {0.0, 0.0};
  int c = 0;
  for (; c + 4 <= nc; c += 4) {
    TP u[2][4], b[2][4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        u[q][k] = partU[(int64_t)(c + k) * mm + e[q]];
        b[q][k] = partB[(int64_t)(c + k) * mm + e[q]];
      }
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        su[q] += (double)u[q][k];
        sb[q] += (double)b[q][k];
      }
  }
  for (; c < nc; ++c)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      su[q] += (double)partU[(int64_t)c * mm + e[q]];
      sb[q] += (double)partB[(int64_t)c * mm + e[q]];
    }
  double v[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const bool off = i[q] != j[q];
    v[q] = 0.0;
    if (in[q]) {
      if (off) v[q] = combine_finish(su[q], sb[q], n_eff, mom ? mom + 2 * e[q] : nullptr);
      else if (mom) mom[2 * e[q]] = mom[2 * e[q] + 1] = 0.0;
      Hr[e[q]] = v[q];
    }
    h[q][ty][tx] = v[q];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 2; ++q)
    if (in[q])
      S[e[q]] = i[q] == j[q] ? 0.0 : (Hx[j[q]] + v[q]) - (Hx[i[q]] + h[1 - q][tx][ty]);
}

}  // namespace vl
