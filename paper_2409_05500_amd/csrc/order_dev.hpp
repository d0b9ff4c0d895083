// Single-wave lookup-only ordering body (Alg. 1 main loop with Eq. 3), shared by the
// single-problem kernel and the batched kernels.
#pragma once
#include <math.h>

#include "common.hpp"

namespace vl {

// ------------------------------------------------------------------------------------------
// Single-wave form for m <= 64 R.  Phase 0: all waves of the block form M0 (this reads every
// row of S once, which also brings S into this CU's L2 for the sequential phase).  Phase 1:
// two waves run the m steps with M in registers and wave-wide minima by DPP / permlane
// butterflies: no barriers inside the sequential loop.  The live set shrinks by one a step, so
// the loop runs in stages of R, R - 1, ..., 1 slots a lane (halving above 8): whenever the live
// entries fit in the next stage's slots they are packed into them through LDS, each slot
// carrying its variable's index.  The packing keeps the indices increasing in (slot, lane)
// order; ties are broken by the index itself, so the result does not depend on the layout.
// ------------------------------------------------------------------------------------------
template <int kCtrl>
__device__ inline double dpp_f64(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  // mov_dpp writes a fresh register (no zeroed "old" operand to set up); the mirror and quad
  // permutations used here give every lane a source lane, so bound_ctrl changes nothing
  return __hiloint2double(__builtin_amdgcn_mov_dpp(hi, kCtrl, 0xF, 0xF, true),
                          __builtin_amdgcn_mov_dpp(lo, kCtrl, 0xF, 0xF, true));
}

template <class T>
__device__ inline T partner16(T v) {
  static_assert(sizeof(T) == 4, "32-bit");
  const unsigned u = __builtin_bit_cast(unsigned, v);
  auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return __builtin_bit_cast(T, ((threadIdx.x >> 4) & 1) ? (unsigned)r[0] : (unsigned)r[1]);
}

template <class T>
__device__ inline T partner32(T v) {
  static_assert(sizeof(T) == 4, "32-bit");
  const unsigned u = __builtin_bit_cast(unsigned, v);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __builtin_bit_cast(T, ((threadIdx.x >> 5) & 1) ? (unsigned)r[0] : (unsigned)r[1]);
}

__device__ inline double partner16_f64(double v) {
  return __hiloint2double(partner16(__double2hiint(v)), partner16(__double2loint(v)));
}
__device__ inline double partner32_f64(double v) {
  return __hiloint2double(partner32(__double2hiint(v)), partner32(__double2loint(v)));
}

// wave-wide minimum (every lane gets it); the lane pairings mirror-in-row, mirror-in-half-row,
// quad xor 2, quad xor 1, xor 16, xor 32 together cover all 64 lanes
__device__ inline double wave_min_f64(double v) {
  v = fmin(v, dpp_f64<kDppRowMirror>(v));
  v = fmin(v, dpp_f64<kDppHalfMirror>(v));
  v = fmin(v, dpp_f64<kDppQuadXor2>(v));
  v = fmin(v, dpp_f64<kDppQuadXor1>(v));
  v = fmin(v, partner16_f64(v));
  v = fmin(v, partner32_f64(v));
  return v;
}

__device__ inline int wave_min_i32(int v) {
  v = min(v, __builtin_amdgcn_mov_dpp(v, kDppRowMirror, 0xF, 0xF, true));
  v = min(v, __builtin_amdgcn_mov_dpp(v, kDppHalfMirror, 0xF, 0xF, true));
  v = min(v, __builtin_amdgcn_mov_dpp(v, kDppQuadXor2, 0xF, 0xF, true));
  v = min(v, __builtin_amdgcn_mov_dpp(v, kDppQuadXor1, 0xF, 0xF, true));
  v = min(v, partner16(v));
  v = min(v, partner32(v));
  return v;
}

// v_min_f64 as written.  fmin() compiles to the same instruction preceded by a v_max_f64 x, x
// per operand (quieting a signalling NaN), one more dependent operation per reduction level;
// the only NaNs here are the quiet ones that mark removed entries, which v_min_f64 passes over.
__device__ __forceinline__ double min_quiet(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

__device__ inline double wave_min_quiet(double v) {
  v = min_quiet(v, dpp_f64<kDppRowMirror>(v));
  v = min_quiet(v, dpp_f64<kDppHalfMirror>(v));
  v = min_quiet(v, dpp_f64<kDppQuadXor2>(v));
  v = min_quiet(v, dpp_f64<kDppQuadXor1>(v));
  v = min_quiet(v, partner16_f64(v));
  v = min_quiet(v, partner32_f64(v));
  return v;
}

// minimum over a lane's R slots (a tree: log2 R dependent steps)
template <int R>
__device__ __forceinline__ double slots_min(const double (&x)[R]) {
  double t[R];
#pragma unroll
  for (int r = 0; r < R; ++r) t[r] = x[r];
#pragma unroll
  for (int s = 1; s < R; s *= 2)
#pragma unroll
    for (int r = 0; r + s < R; r += 2 * s) t[r] = min_quiet(t[r], t[r + s]);
  return t[0];
}

// lowest index among a lane's slots holding key (2^31 - 1 when none)
template <int R>
__device__ __forceinline__ int slots_index_of(const double (&x)[R], const int (&vid)[R],
                                              double key) {
  int t[R];
#pragma unroll
  for (int r = 0; r < R; ++r) t[r] = x[r] == key ? vid[r] : 0x7fffffff;
#pragma unroll
  for (int s = 1; s < R; s *= 2)
#pragma unroll
    for (int r = 0; r + s < R; r += 2 * s) t[r] = min(t[r], t[r + s]);
  return t[0];
}

// The wave's smallest key (NaN: none) and, in lane, the one lane that holds it, or -1 where several
// may: the wave compares the high words only, as ordered integers (one operation a level, where
// an FP64 minimum takes two moves and one); equal high words (equal or nearly equal keys, or
// none) take the full reduction.
__device__ __forceinline__ double wave_lowest(double key, int& lane) {
  const int hi = __double2hiint(key);
  const int hk = key == key ? hi ^ ((hi >> 31) & 0x7fffffff) : 0x7fffffff;
  int v = hk;
  v = min(v, __builtin_amdgcn_mov_dpp(v, kDppRowMirror, 0xF, 0xF, true));
  v = min(v, __builtin_amdgcn_mov_dpp(v, kDppHalfMirror, 0xF, 0xF, true));
  v = min(v, __builtin_amdgcn_mov_dpp(v, kDppQuadXor2, 0xF, 0xF, true));
  v = min(v, __builtin_amdgcn_mov_dpp(v, kDppQuadXor1, 0xF, 0xF, true));
  const int low = min(min(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
                      min(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
  const unsigned long long mk = __ballot(hk == low);
  lane = -1;
  if (__builtin_expect((mk & (mk - 1)) != 0, 0)) return wave_min_quiet(key);
  lane = __builtin_ctzll(mk);
  return __hiloint2double(__builtin_amdgcn_readlane(hi, lane),
                          __builtin_amdgcn_readlane(__double2loint(key), lane));
}

// Which part of a step a wave does: all of it, or one of two waves' shares.
enum class OrderRole { kAll, kOrder, kMargin };

// What the ordering wave tells the margin wave of each step, in LDS: index is written last (-1:
// not yet), and a wave's LDS accesses are carried out in order.
template <int N>
struct OrderBox {
  double low[N];
  int index[N];
};

constexpr int order_next_slots(int R) { return R > 8 ? R / 2 : R - 1; }

// Steps k .. while more entries are live than the next stage holds, with R slots a lane
// (Mv[r], vid[r]: the lane's entries and their variable indices; removed and empty slots hold
// NaN).  Removed and padding entries hold NaN: the minimum passes over NaN, and NaN equals
// nothing, so they never win a minimum nor the index search even when every live M is +inf (a
// row of S with a non-finite entry, which raised VL_ERR_NONFINITE).  A step finds the smallest M
// (m1) and the lowest index that holds it (i1), loads row i1 of S and updates M by it; its margin
// is the smallest M left without i1.  It costs one wave's dependent instructions (8 cycles and
// more each), so with few slots what the next step does not need is another wave's: the ordering
// wave posts m1 and i1, and the margin wave, with an M of its own, takes each post, which always
// comes, and does the rest.  Where the slots' own work is the most of it (R > 8) one wave does
// all, the margin's reduction while the row is loaded.  The results are stored 64 steps at a
// time: the wait for a row counts every memory operation of the wave, so a step that stores
// waits for its stores.  In us, with one wave that stores at each step and reduces FP64 values
// throughout, and now: m = 100 49 and 38, m = 317 183 and 152, m = 1000 (with its B0 and lag
// matrices) 1312 and 1231.  sM, sI: LDS for the packing, the wave's own (64 RN entries each).
template <int R, OrderRole kRole, int N>
__device__ __forceinline__ void order_stage(const double* S, int64_t m,
                                            int32_t* __restrict__ order,
                                            double* __restrict__ margin, OrderBox<N>& box,
                                            double* sM, int* sI, double (&Mv)[R], int (&vid)[R],
                                            int k, int out_i, double out_m) {
  const int lane = threadIdx.x & 63;
  const double inf = INFINITY, gone = __builtin_nan("");
  const int last = (int)m - 1;
  constexpr int RN = order_next_slots(R);
  const int kend = RN > 0 ? (int)m - 64 * RN : (int)m;   // m - k entries are live at step k
  for (; k < kend; ++k) {
    double m1;
    int i1;
    if constexpr (kRole == OrderRole::kMargin) {
      volatile int* post = &box.index[k];
      do i1 = *post;
      while (i1 < 0);
      i1 = __builtin_amdgcn_readfirstlane(i1);
      m1 = *(volatile double*)&box.low[k];
    } else {
      const double key = slots_min<R>(Mv);
      const int own = slots_index_of<R>(Mv, vid, key);
      int l;
      m1 = wave_lowest(key, l);
      if (__builtin_expect(l >= 0, 1)) i1 = __builtin_amdgcn_readlane(own, l);
      else i1 = __builtin_amdgcn_readfirstlane(wave_min_i32(key == m1 ? own : 0x7fffffff));
    }
    // row i1 of S at this lane's variables (every vid is a valid column)
    const double* rowp = S + (unsigned)min(i1, last) * (unsigned)m;
    double v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = rowp[vid[r]];
    if constexpr (kRole == OrderRole::kOrder) {
      if (lane == 0) {
        *(volatile double*)&box.low[k] = m1;
        *(volatile int*)&box.index[k] = i1;
      }
    }
    // remove the winner (any low word with this high word is a NaN)
#pragma unroll
    for (int r = 0; r < R; ++r)
      Mv[r] = __hiloint2double(vid[r] == i1 ? 0x7ff80000 : __double2hiint(Mv[r]),
                               __double2loint(Mv[r]));
    if constexpr (kRole != OrderRole::kOrder) {
      int l;
      const double m2 = wave_lowest(slots_min<R>(Mv), l);    // NaN when no live entry is left
      const double gap = (m2 == inf || m2 != m2) ? inf : m2 - m1;
      const bool mine = lane == (k & 63);
      out_i = mine ? i1 : out_i;
      out_m = mine ? gap : out_m;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      // 0 for v <= 0, NaN and infinity (a zero high word leaves a number whose square is 0)
      const bool up = v[r] > 0.0 && v[r] < inf;
      const double pos = __hiloint2double(up ? __double2hiint(v[r]) : 0, __double2loint(v[r]));
      Mv[r] -= pos * pos;            // +inf stays +inf, NaN stays NaN
    }
    if constexpr (kRole != OrderRole::kOrder) {
      if ((k & 63) == 63 || k == last) {
        const int ko = (k & ~63) + lane;
        if (ko <= k) {
          order[ko] = out_i;
          margin[ko] = out_m;
        }
      }
    }
  }
  if constexpr (RN > 0) {
    // pack the live entries into RN slots: position = live entries before this one in (slot,
    // lane) order, from one ballot per slot (the wave writes, then reads, its own LDS)
    int base = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const bool live = Mv[r] == Mv[r];
      const unsigned long long mk = __ballot(live);
      const int pos = base + __builtin_popcountll(mk & ((1ull << lane) - 1ull));
      if (live) {
        sM[pos] = Mv[r];
        sI[pos] = vid[r];
      }
      base += __builtin_popcountll(mk);
    }
    double Mn[RN];
    int vn[RN];
#pragma unroll
    for (int r = 0; r < RN; ++r) {
      const int p = lane + 64 * r;
      Mn[r] = p < base ? sM[p] : gone;
      vn[r] = p < base ? sI[p] : 0;
    }
    order_stage<RN, kRole>(S, m, order, margin, box, sM, sI, Mn, vn, k, out_i, out_m);
  }
}

// kLds: S is first copied to LDS (m <= 64 R; 64 R squared doubles), a shorter wait for each row
template <int R, int kThreads, bool kLds = false>
__device__ __forceinline__ void order_wave_block(const double* __restrict__ Sg, int64_t m,
                                        int32_t* __restrict__ order, double* __restrict__ margin,
                                        int32_t* st) {
  __shared__ double M0s[64 * R];   // M0
  constexpr int kPack = 64 * (order_next_slots(R) > 0 ? order_next_slots(R) : 1);
  constexpr bool kTwo = R <= 8;    // an ordering and a margin wave, else one wave without a mailbox
  __shared__ double packM[kTwo ? 2 : 1][kPack];
  __shared__ int packI[kTwo ? 2 : 1][kPack];
  __shared__ OrderBox<kTwo ? 64 * R : 1> box;
  __shared__ double Sl[kLds ? 64 * R * 64 * R : 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if constexpr (kLds) {
    constexpr int kF = 8;
    const int total = (int)(m * m);
    for (int e0 = threadIdx.x; e0 < total; e0 += kF * kThreads) {
      double v[kF];
#pragma unroll
      for (int q = 0; q < kF; ++q) {
        const int e = e0 + q * kThreads;
        v[q] = Sg[e < total ? e : total - 1];
      }
#pragma unroll
      for (int q = 0; q < kF; ++q)
        if (e0 + q * kThreads < total) Sl[e0 + q * kThreads] = v[q];
    }
    __syncthreads();
  }
  const double* S = Sg;
  if constexpr (kLds) S = Sl;
  bool bad = false;
  // several rows per wave at once, every load of them issued before the sums (clamped
  // in-bounds addresses; the padding is skipped in the sums)
  constexpr int kRows = R <= 4 ? 4 : (R <= 8 ? 2 : 1);
  for (int64_t row0 = (int64_t)wave * kRows; row0 < m; row0 += (int64_t)(kThreads / 64) * kRows) {
    double v[kRows][R];
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
      const int64_t row = row0 + q < m ? row0 + q : m - 1;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int64_t j = lane + 64 * r;
        v[q][r] = S[row * m + (j < m ? j : m - 1)];
      }
    }
#pragma unroll
    for (int q = 0; q < kRows; ++q) {
      const int64_t row = row0 + q;
      double s = 0.0;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int64_t j = lane + 64 * r;
        const bool in = j < m && row < m;
        bad |= in && !isfinite(v[q][r]);
        if (in && j != row && v[q][r] < 0.0) s += v[q][r] * v[q][r];
      }
      s = wave_sum_d(s);
      if (lane == 0 && row < m) M0s[row] = isfinite(s) ? s : INFINITY;
    }
  }
  if (bad) raise_status(st, VL_ERR_NONFINITE);
  if constexpr (kTwo)
    for (int e = threadIdx.x; e < (int)m; e += kThreads) box.index[e] = -1;
  __syncthreads();
  static_assert(kThreads >= 128, "an ordering and a margin wave");
  if (wave < (kTwo ? 2 : 1)) {
    const double gone = __builtin_nan("");
    double Mv[R];
    int vid[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = lane + 64 * r;
      Mv[r] = i < m ? M0s[i] : gone;
      vid[r] = i < m ? i : 0;
    }
    if constexpr (!kTwo)
      order_stage<R, OrderRole::kAll>(S, m, order, margin, box, packM[0], packI[0], Mv, vid, 0, 0,
                                      0.0);
    else if (wave == 0)
      order_stage<R, OrderRole::kOrder>(S, m, order, margin, box, packM[0], packI[0], Mv, vid, 0, 0,
                                        0.0);
    else
      order_stage<R, OrderRole::kMargin>(S, m, order, margin, box, packM[1], packI[1], Mv, vid, 0,
                                         0, 0.0);
  }
  __syncthreads();
}

}  // namespace vl
