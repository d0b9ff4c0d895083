// Residual GEMM tiles of the VAR fit, shared by the single-problem and batched kernels.
// Y = x(t) and Z = [x(t-1), ..., x(t-p)] are read through the column map of the lagged views
// (colmap[tau m + i] = offset of x_i(t - tau) at t = 0), centred by mu (same layout).
#pragma once
#include "common.hpp"

namespace vl {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// E[t][j] = (Y(t,j) - muY[j]) - sum_k (Z(t,k) - muZ[k]) CoefF[k][j]
// Block tile 64 (t) x 64 (j), 4 waves of 32 x 32, v_mfma_f32_32x32x2f32, k step 32 via LDS.
__device__ inline void var_residual_tile_f32(
    const float* __restrict__ X, int64_t ldx, const int64_t* __restrict__ colmap,
    const double* __restrict__ mu, int64_t m, int p, int64_t n_eff,
    const float* __restrict__ CoefF, float* __restrict__ E, int64_t lde, int64_t t0,
    int64_t j0) {
  __shared__ float Zs[32][64 + 1];
  __shared__ float Cs[32][64 + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wi = wave >> 1, wj = wave & 1;
  const int64_t dz = m * p;
  const int64_t* mapZ = colmap + m;
  const double* muZ = mu + m;
  f32x16 acc = {};
  // the output column's offset and mean, read before the products
  const int64_t jo = j0 + wj * 32 + (lane & 31);
  const int64_t offy = colmap[jo < m ? jo : 0];
  const float muy = (float)mu[jo < m ? jo : 0];
  for (int64_t k0 = 0; k0 < dz; k0 += 32) {
    {
      const int kk = tid & 31, tt = tid >> 5;
      const int64_t k = k0 + kk;
      const bool vk = k < dz;
      // clamped in-bounds addresses, padding masked after the loads (no branch per load)
      const int64_t off = mapZ[vk ? k : dz - 1];
      const float mz = vk ? (float)muZ[k] : 0.f;
      float xv[8], cv[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const int64_t t = t0 + tt + 8 * r;
        xv[r] = X[off + (t < n_eff ? t : n_eff - 1) * ldx];
      }
      const int jj = tid & 63, kr = tid >> 6;
      const int64_t jc = j0 + jj < m ? j0 + jj : m - 1;
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const int64_t kq = k0 + kr + 4 * r;
        cv[r] = CoefF[(kq < dz ? kq : dz - 1) * m + jc];
      }
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const int64_t t = t0 + tt + 8 * r;
        Zs[kk][tt + 8 * r] = mask_f32(xv[r] - mz, vk && t < n_eff);
      }
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const int64_t kq = k0 + kr + 4 * r;
        Cs[kr + 4 * r][jj] = mask_f32(cv[r], kq < dz && j0 + jj < m);
      }
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 32; kk += 2) {
      const float a = Zs[kk + (lane >> 5)][wi * 32 + (lane & 31)];
      const float b = Cs[kk + (lane >> 5)][wj * 32 + (lane & 31)];
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
    }
    __syncthreads();
  }
  // Y at this lane's outputs: every load issued before the first store (clamped addresses;
  // a load under each store's bounds test would wait for each in turn)
  float yin[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int64_t t = t0 + wi * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    yin[r] = X[offy + (t < n_eff ? t : n_eff - 1) * ldx];
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int64_t t = t0 + wi * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    if (t < n_eff && jo < m) E[t * lde + jo] = (yin[r] - muy) - acc[r];
  }
}

// FP64 variant of the residual GEMM, one wave: 16 NA samples x 16 NB variables by
// v_mfma_f64_16x16x4f64 on the widened, centred FP32 lags and the FP64 coefficients (exact
// products, FP64 sums; E is rounded once, at the end).  Both operands come straight from memory in
// the products' own layout, sixteen lags a step: a lane holds four consecutive lags of its sample
// and the four products of a step take one of each lane's, so the coefficients of lag
// 4 (l / 16) + s go with product s.  No LDS, no barrier, waves past the samples leave.
// This form takes any size; var_residual_wide_f64 is the one for the bulk of the work.
template <int NA, int NB>
__device__ __forceinline__ void var_residual_wave_f64(
    const float* __restrict__ X, int64_t ldx, const int64_t* __restrict__ colmap,
    const double* __restrict__ mu, int64_t m, int p, int64_t n_eff,
    const double* __restrict__ Coef, float* __restrict__ E, int64_t lde, int64_t t0, int64_t j0) {
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  if (t0 >= n_eff || j0 >= m) return;
  // live 16-wide blocks; samples and variables past the edge read the last one
  const int na = (int)(n_eff - t0 < 16 * NA ? (n_eff - t0 + 15) / 16 : NA);
  const int nb = (int)(m - j0 < 16 * NB ? (m - j0 + 15) / 16 : NB);
  const float* px[NA];
  int jq[NB];
#pragma unroll
  for (int a = 0; a < NA; ++a) {
    const int64_t t = t0 + 16 * a + li;
    px[a] = X + (t < n_eff ? t : n_eff - 1) * ldx;
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int64_t j = j0 + 16 * b + li;
    jq[b] = (int)(j < m ? j : m - 1);
  }
  f64x4 acc[NA][NB];
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
  float x[NA][4];
  double mz[4], cf[4][NB];
  const int mi = (int)m;
  // lags i0 .. i0 + 15 of lag block tau (wave-uniform); past the block's end the last variable's
  // values with zero coefficients
  auto load = [&](int tau, int i0) {
    const int64_t off = colmap[(int64_t)tau * m];
    const double* mt = mu + (int64_t)tau * m;
    const double* ct = Coef + (int64_t)(tau - 1) * m * m;
    const int i = i0 + 4 * lk;
    if (i0 + 16 <= mi) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
#pragma unroll
        for (int a = 0; a < NA; ++a) x[a][s] = px[a][off + i + s];
        mz[s] = mt[i + s];
#pragma unroll
        for (int b = 0; b < NB; ++b) cf[s][b] = ct[(i + s) * mi + jq[b]];
      }
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int is = i + s < mi ? i + s : mi - 1;
#pragma unroll
        for (int a = 0; a < NA; ++a) x[a][s] = px[a][off + is];
        mz[s] = mt[is];
#pragma unroll
        for (int b = 0; b < NB; ++b) cf[s][b] = mask_f64(ct[is * mi + jq[b]], i + s < mi);
      }
    }
  };
  int tau = 1, i0 = 0;
  load(tau, i0);
  for (;;) {
    double av[4][NA], bv[4][NB];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
#pragma unroll
      for (int a = 0; a < NA; ++a) av[s][a] = (double)x[a][s] - mz[s];
#pragma unroll
      for (int b = 0; b < NB; ++b) bv[s][b] = cf[s][b];
    }
    i0 += 16;
    if (i0 >= mi) {
      i0 = 0;
      ++tau;
    }
    const bool more = tau <= p;
    if (more) load(tau, i0);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int a = 0; a < NA; ++a)
        if (a < na) {
#pragma unroll
          for (int b = 0; b < NB; ++b)
            if (b < nb)
              acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[s][a], bv[s][b], acc[a][b], 0, 0, 0);
        }
    if (!more) break;
  }
  // Y at this lane's outputs, a block row at a time: its loads issued before its stores
  double muy[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) muy[b] = mu[jq[b]];
#pragma unroll
  for (int a = 0; a < NA; ++a) {
    float y[NB][4];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t t = t0 + a * 16 + lk + 4 * r;                   // f64 D layout
        y[b][r] = X[colmap[0] + jq[b] + (t < n_eff ? t : n_eff - 1) * ldx];
      }
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t t = t0 + a * 16 + lk + 4 * r, j = j0 + b * 16 + li;
        if (t < n_eff && j < m) E[t * lde + j] = (float)(((double)y[b][r] - muy[b]) - acc[a][b][r]);
      }
  }
}

// The same for 64 samples x 16 NB variables where n_eff >= 64 and m >= 16, without a test in the
// loop: the last samples and the last lags of a block are taken as a whole group that overlaps the
// one before (the same values written twice; the lags seen before count as zero), so every load
// is a full one (a lane's four lags in one, whatever their alignment) and can be counted.  A step
// converts its sixteen lags first, then loads the next sixteen, and each product's coefficients
// are loaded again as soon as it has used them.  sums[j]: the stored E of column j added up over the
// samples from t0 on (those no other tile has), for the column means.  Bound by the FP64 matrix rate, two waves per
// SIMD, and by the memory for Y and E at the end.  Against 64 x 64 tiles staged in LDS, four
// waves a tile: 256 problems (m 20-200, n 500-8000) 1136 -> 824 us, 181 windows of 50 x 2000
// 102 -> 77.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

template <int NB>
__device__ __forceinline__ void var_residual_wide_f64(
    const float* __restrict__ X, int64_t ldx, const double* __restrict__ mu, int m, int p,
    int64_t n_eff, const double* __restrict__ Coef, float* __restrict__ E, int64_t lde, int64_t t0,
    int j0, double* __restrict__ sums) {
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int64_t tnew = t0;
  t0 = t0 < n_eff - 64 ? t0 : n_eff - 64;
  int jq[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) jq[b] = j0 + 16 * b + li < m ? j0 + 16 * b + li : m - 1;
  const float* px = X + (t0 + li) * ldx + 4 * lk;
  f64x4 acc[4][NB];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
  f32x4u x[4];
  double mz[4], cf[4][NB];
  const int groups = (m + 15) / 16;                  // of a lag block
  // group g of lag block tau: lags ia .. ia + 15, those from 16 g on new
  auto first = [&](int g) { return 16 * g + 16 <= m ? 16 * g : m - 16; };
  auto load_x = [&](int tau, int g) {
    const int ia = first(g);
    const float* q = px + (p - tau) * ldx + ia;
#pragma unroll
    for (int a = 0; a < 4; ++a) x[a] = *reinterpret_cast<const f32x4u*>(q + 16 * a * ldx);
#pragma unroll
    for (int s = 0; s < 4; ++s) mz[s] = mu[tau * m + ia + 4 * lk + s];
  };
  auto load_c = [&](int tau, int g, int s) {
    const double* c = Coef + ((tau - 1) * m + first(g) + 4 * lk + s) * m;
#pragma unroll
    for (int b = 0; b < NB; ++b) cf[s][b] = c[jq[b]];
  };
  load_x(1, 0);
#pragma unroll
  for (int s = 0; s < 4; ++s) load_c(1, 0, s);
  __builtin_amdgcn_sched_barrier(0);
  int tau = 1, g = 0;
  for (int left = p * groups; left > 0; --left) {
    const int seen = 16 * g - first(g);              // lags of this group counted before
    int taun = tau, gn = g;
    if (left > 1) {                                  // (past the end: the last group again)
      gn = g + 1 < groups ? g + 1 : 0;
      taun = gn == 0 ? tau + 1 : tau;
    }
    double av[4][4];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        av[s][a] = mask_f64((double)x[a][s] - mz[s], 4 * lk + s >= seen);
        asm volatile("" : "+v"(av[s][a]));           // formed here, not at each product
      }
    load_x(taun, gn);
    __builtin_amdgcn_sched_barrier(0);               // (loads stay in this order)
#pragma unroll
    for (int s = 0; s < 4; ++s) {
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[s][a], cf[s][b], acc[a][b], 0, 0, 0);
      load_c(taun, gn, s);
      __builtin_amdgcn_sched_barrier(0);
    }
    tau = taun;
    g = gn;
  }
  // Y at this lane's outputs, a block row at a time: its loads issued before its stores
  double muy[NB], total[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    muy[b] = mu[jq[b]];
    total[b] = 0.0;
  }
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const int64_t t = t0 + 16 * a + lk;              // f64 D layout: rows lk + 4 r
    float y[NB][4];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) y[b][r] = X[(t + 4 * r + p) * ldx + jq[b]];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float e = (float)(((double)y[b][r] - muy[b]) - acc[a][b][r]);
        if (j0 + 16 * b + li < m) E[(t + 4 * r) * lde + jq[b]] = e;
        total[b] += mask_f64((double)e, t + 4 * r >= tnew);
      }
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    total[b] += __shfl_xor(total[b], 16, 64);
    total[b] += __shfl_xor(total[b], 32, 64);
    if (lk == 0 && j0 + 16 * b + li < m) sums[jq[b]] = total[b];
  }
}

// ------------------------------------------------------------------------------------------
// FP64 residual tile: RT samples x 64 variables per workgroup; wave (wi, wj) of the 2 x 2 waves
// owns RT/2 x 32 = RT/32 x 2 blocks of v_mfma_f64_16x16x4f64.  Stages of RK lags through LDS
// (the centred lag values widened to FP64 once, at load); the next stage's global loads are in
// flight during the products.  Every output element sums its products in lag order four at a
// time whatever RT and RK, so all shapes give the same bits.
// ------------------------------------------------------------------------------------------
constexpr int kRJ = 64;        // variables per tile

template <class TOut, int RT, int RK>
__device__ inline void var_residual_tile_f64w(
    const float* __restrict__ X, int64_t ldx, const int64_t* __restrict__ colmap,
    const double* __restrict__ mu, int64_t m, int p, int64_t n_eff,
    const double* __restrict__ Coef, TOut* __restrict__ E, int64_t lde, int64_t t0, int64_t j0) {
  constexpr int XB = RT / 32;                  // 16-row blocks per wave
  __shared__ double Zs[RK][RT + 1];
  __shared__ double Cs[RK][kRJ + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wi = wave >> 1, wj = wave & 1, li = lane & 15, lk = lane >> 4;
  const int64_t dz = m * p;
  const int64_t* mapZ = colmap + m;
  const double* muZ = mu + m;
  f64x4 acc[XB][2];
#pragma unroll
  for (int x = 0; x < XB; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = f64x4{0.0, 0.0, 0.0, 0.0};
  constexpr int kZRows = 256 / RK;             // Z loader: RK lags x kZRows sample rows a pass
  constexpr int kZPass = RT / kZRows;
  const int zk = tid % RK, zt = tid / RK;
  const int cj = tid & 63, ck = tid >> 6;      // Coef loader: 64 variables x 4 lags per pass
  double rz[kZPass], rc[RK / 4];
  // Every load reads a clamped in-bounds address and the padding is selected afterwards, so
  // the loads of a stage issue back to back (no branch, no wait per load).
  const int64_t jc = j0 + cj < m ? j0 + cj : m - 1;
  const bool vj = j0 + cj < m;
  auto load = [&](int64_t k0) {
    const int64_t k = k0 + zk;
    const bool vk = k < dz;
    const int64_t off = mapZ[vk ? k : dz - 1];
    const double mz = vk ? muZ[k] : 0.0;
    float xv[kZPass];
#pragma unroll
    for (int u = 0; u < kZPass; ++u) {
      const int64_t t = t0 + zt + kZRows * u;
      xv[u] = X[off + (t < n_eff ? t : n_eff - 1) * ldx];
    }
#pragma unroll
    for (int u = 0; u < RK / 4; ++u) {
      const int64_t kq = k0 + ck + 4 * u;
      const double cv = Coef[(kq < dz ? kq : dz - 1) * m + jc];
      rc[u] = mask_f64(cv, kq < dz && vj);
    }
#pragma unroll
    for (int u = 0; u < kZPass; ++u) {
      const int64_t t = t0 + zt + kZRows * u;
      rz[u] = mask_f64((double)xv[u] - mz, vk && t < n_eff);
    }
  };
  load(0);
  for (int64_t k0 = 0; k0 < dz; k0 += RK) {
#pragma unroll
    for (int u = 0; u < kZPass; ++u) Zs[zk][zt + kZRows * u] = rz[u];
#pragma unroll
    for (int u = 0; u < RK / 4; ++u) Cs[ck + 4 * u][cj] = rc[u];
    __syncthreads();
    if (k0 + RK < dz) load(k0 + RK);
#pragma unroll
    for (int kk = 0; kk < RK; kk += 4) {
      double a[XB], b[2];
#pragma unroll
      for (int x = 0; x < XB; ++x) a[x] = Zs[kk + lk][wi * (RT / 2) + x * 16 + li];
#pragma unroll
      for (int y = 0; y < 2; ++y) b[y] = Cs[kk + lk][wj * 32 + y * 16 + li];
#pragma unroll
      for (int x = 0; x < XB; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
          acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[x], b[y], acc[x][y], 0, 0, 0);
    }
    __syncthreads();
  }
  // Y at this lane's outputs: every load issued before the first store (clamped addresses)
  float yin[XB][2][4];
#pragma unroll
  for (int y = 0; y < 2; ++y) {
    const int64_t j = j0 + wj * 32 + y * 16 + li;
    const int64_t offy = colmap[j < m ? j : 0];
#pragma unroll
    for (int x = 0; x < XB; ++x)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t t = t0 + wi * (RT / 2) + x * 16 + lk + 4 * r;     // f64 D layout
        yin[x][y][r] = X[offy + (t < n_eff ? t : n_eff - 1) * ldx];
      }
  }
#pragma unroll
  for (int y = 0; y < 2; ++y) {
    const int64_t j = j0 + wj * 32 + y * 16 + li;
    const double muy = mu[j < m ? j : 0];
#pragma unroll
    for (int x = 0; x < XB; ++x)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t t = t0 + wi * (RT / 2) + x * 16 + lk + 4 * r;
        if (t < n_eff && j < m) E[t * lde + j] = (TOut)(((double)yin[x][y][r] - muy) - acc[x][y][r]);
      }
  }
}

}  // namespace vl
