// The original iterative DirectLiNGAM ordering (Sec. 3 steps 1-5), the search that the
// heuristic's one-time precompute replaces.  Each step scores every ordered pair of the
// remaining variables on the current data (the pairwise stage of the heuristic path, on the
// current columns), picks the variable with the smallest aggregate M_i = sum_j min(0, S_ij)^2
// (Eq. 3; lowest index on exact ties), then replaces every remaining column by its residual on
// the pick, computed from the standardised columns (Sec. 3 step 5):
//     x_j <- (x_j - mu_j)/s_j - rho_jc (x_c - mu_c)/s_c,
// and drops the pick.  The current columns stay in ascending original order (a compacting
// copy), so the lowest current index is the lowest original index.  One pairwise pass per step:
// sum_u u^2 n = O(m^3 n) sample-evals in all.  The loop is launched from the host without
// synchronisation: the pick stays on the device.
#include "iterative.hpp"
#include "gram.hpp"
#include "order.hpp"
#include "pairwise.hpp"
#include "profile.hpp"

#include <algorithm>

namespace vl {

__global__ void iter_init_kernel(int32_t* __restrict__ idx, int64_t m) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < m) idx[e] = (int32_t)e;
}

constexpr int kIterMaxM = 4096;

// M_i over the u current columns, the pick c (smallest M, lowest index on ties) and the margin
// (second-smallest M minus the smallest; +inf with one column left).  One workgroup: its threads
// are split over slices of each column, so a step's whole S is a load or two a thread, and the
// argmin runs in registers (one thread a column and a tree over LDS for each minimum: 6.5 us a
// step at m = 100, this 6.0; with 1024 threads 8.8).
constexpr int kSelThreads = 256;

struct IterBest {
  double m1, m2;
  int i1;
};

__device__ inline IterBest iter_better(IterBest a, IterBest b) {
  const bool w = b.m1 < a.m1 || (b.m1 == a.m1 && b.i1 < a.i1);
  IterBest r;
  r.m1 = w ? b.m1 : a.m1;
  r.i1 = w ? b.i1 : a.i1;
  r.m2 = fmin(w ? a.m1 : b.m1, w ? b.m2 : a.m2);
  return r;
}

__global__ __launch_bounds__(kSelThreads) void iter_select_kernel(
    const double* __restrict__ S, int64_t u, const int32_t* __restrict__ idx, int64_t k,
    int32_t* __restrict__ order, double* __restrict__ margin, int32_t* __restrict__ pick) {
  __shared__ double part[kSelThreads];
  __shared__ IterBest wbest[kSelThreads / 64];
  const int tid = threadIdx.x;
  if (u == 1) {
    if (tid == 0) {
      order[k] = idx[0];
      margin[k] = INFINITY;
      *pick = 0;
    }
    return;
  }
  int width = 64;                                    // threads over the columns
  while (width < u && width < kSelThreads) width <<= 1;
  const int slices = kSelThreads / width;            // of a column's rows (1 from u = 129 on)
  const int64_t len = ceil_div(u, (int64_t)slices);
  const int64_t j0 = (tid / width) * len, j1 = j0 + len < u ? j0 + len : u;
  IterBest best{INFINITY, INFINITY, 0x7fffffff};
  // S is antisymmetric bit for bit (S_ji = -S_ij), so min(0, S_ij)^2 = max(0, S_ji)^2: read along
  // columns (consecutive threads, consecutive words), 32 loads in flight, the last group's from
  // clamped addresses
  constexpr int kL = 32;
  for (int64_t i = tid & (width - 1); i < u; i += width) {
    double s = 0.0;
    for (int64_t j = j0; j < j1; j += kL) {
      double v[kL];
#pragma unroll
      for (int q = 0; q < kL; ++q) v[q] = S[(j + q < j1 ? j + q : j1 - 1) * u + i];
#pragma unroll
      for (int q = 0; q < kL; ++q)
        if (j + q < j1 && j + q != i && v[q] > 0.0) s += v[q] * v[q];
    }
    part[tid] = s;
    if (slices == 1) best = iter_better(best, IterBest{s, INFINITY, (int)i});
  }
  if (slices > 1) {
    __syncthreads();
    if (tid < u) {
      double s = part[tid];
      for (int q = 1; q < slices; ++q) s += part[q * width + tid];
      best = IterBest{s, INFINITY, tid};
    }
  }
#pragma unroll
  for (int h = 32; h > 0; h >>= 1)
    best = iter_better(best, IterBest{__shfl_xor(best.m1, h, 64), __shfl_xor(best.m2, h, 64),
                                      __shfl_xor(best.i1, h, 64)});
  if ((tid & 63) == 0) wbest[tid >> 6] = best;
  __syncthreads();
  if (tid == 0) {
    for (int q = 1; q < kSelThreads / 64; ++q) best = iter_better(best, wbest[q]);
    const int c = best.i1 < u ? best.i1 : 0;
    order[k] = idx[c];
    margin[k] = best.m2 - best.m1;
    *pick = c;
  }
}

// Column j' of the next data: the standardised x_j minus rho_jc times the standardised x_c,
// with j = j' + (j' >= c); FP64 arithmetic, FP32 storage.  The grid is colmeans()'s, 64 columns by
// a split of the rows, four row lanes: the splits' sums of the stored columns come out of the same
// pass, in the same order, for the next step's means (in two launches 8.0 us a step at m = 100,
// n = 5000; in this one 5.6, with the rows' pointers stepped: 64-bit address products for each
// load took it to 8.3).
__global__ __launch_bounds__(256) void iter_refine_kernel(
    const float* __restrict__ Ek, int64_t ldk, int64_t n_eff, int64_t u,
    const double* __restrict__ mu, const double* __restrict__ Cov,
    const int32_t* __restrict__ pick, const int32_t* __restrict__ idx_in,
    int32_t* __restrict__ idx_out, float* __restrict__ En, int64_t ldn, int64_t rows_per_split,
    double* __restrict__ part) {
  __shared__ double red[4][64];
  const int cc = threadIdx.x & 63, rg = threadIdx.x >> 6;
  const int64_t w = u - 1, jp = (int64_t)blockIdx.x * 64 + cc;
  const int64_t r0 = (int64_t)blockIdx.y * rows_per_split;
  const int64_t r1 = r0 + rows_per_split < n_eff ? r0 + rows_per_split : n_eff;
  double s = 0.0;
  if (jp < w) {
    const int64_t c = *pick;
    const int64_t j = jp + (jp >= c ? 1 : 0);
    const double sj = sqrt(Cov[j * u + j]), muj = mu[j];
    const double sc = sqrt(Cov[c * u + c]), muc = mu[c];
    const double ij = 1.0 / sj, rc = Cov[j * u + c] / (sj * sc) / sc;
    constexpr int kF = 8;                            // rows in flight, in row order
    const int64_t step = 4 * ldk, nstep = 4 * ldn;
    const float* pj = Ek + (r0 + rg) * ldk + j;
    const float* pc = Ek + (r0 + rg) * ldk + c;
    float* pn = En + (r0 + rg) * ldn + jp;
    auto put = [&](float ej, float ec) {
      const float f = (float)(((double)ej - muj) * ij - rc * ((double)ec - muc));
      *pn = f;
      pn += nstep;
      s += (double)f;
    };
    int64_t t = r0 + rg;
    for (; t + 4 * (kF - 1) < r1; t += 4 * kF) {
      float ej[kF], ec[kF];
#pragma unroll
      for (int q = 0; q < kF; ++q, pj += step, pc += step) {
        ej[q] = *pj;
        ec[q] = *pc;
      }
#pragma unroll
      for (int q = 0; q < kF; ++q) put(ej[q], ec[q]);
    }
    for (; t < r1; t += 4, pj += step, pc += step) put(*pj, *pc);
    if (blockIdx.y == 0 && rg == 0) idx_out[jp] = idx_in[j];
  }
  red[rg][cc] = s;
  __syncthreads();
  if (rg == 0 && jp < w)
    part[(int64_t)blockIdx.y * w + jp] = ((red[0][cc] + red[1][cc]) + red[2][cc]) + red[3][cc];
}

// Hybrid finish: the remaining variables' lookup order, mapped to original indices.
__global__ void iter_map_kernel(const int32_t* __restrict__ osub,
                                const int32_t* __restrict__ idx, int64_t u,
                                int32_t* __restrict__ order) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= u) return;
  int32_t v = osub[r];
  v = v < 0 ? 0 : (v >= u ? (int32_t)u - 1 : v);
  order[r] = idx[v];
}

size_t iter_ws_bytes(int64_t n_eff, int64_t m, void* base, IterWs* out) {
  Carver c(base);
  IterWs w;
  w.D[0] = c.take<float>(n_eff * m);
  w.D[1] = c.take<float>(n_eff * m);
  w.idx[0] = c.take<int32_t>(m);
  w.idx[1] = c.take<int32_t>(m);
  w.pick = c.take<int32_t>(1);
  w.Hx = c.take<double>(m);
  w.Hr = c.take<double>(m * m);
  w.S = c.take<double>(m * m);
  w.Cov = c.take<double>(m * m);
  size_t pw = 0;
  for (int64_t u = 2; u <= m; ++u)
    pw = std::max(pw, pairwise_ws_bytes(plan_pairwise(n_eff, u), nullptr, nullptr));
  w.pw = c.take<char>(pw);
  w.osub = c.take<int32_t>(m);
  w.M0 = c.take<double>(m);
  if (out) *out = w;
  return c.used;
}

int run_order_iterative(const float* E, int64_t n_eff, int64_t m, int64_t lde, int prec,
                        int64_t k_exact, int32_t* order, double* margin, const IterWs& w,
                        int32_t* st, hipStream_t stream) {
  if (m > kIterMaxM) return VL_ERR_SHAPE;
  ProfileScope ps("iterative", stream);
  iter_init_kernel<<<(unsigned)ceil_div(m, (int64_t)256), 256, 0, stream>>>(w.idx[0], m);
  VL_LAUNCH_CHECK();
  const float* cur = E;
  int64_t ldc = lde;
  for (int64_t k = 0; k < m; ++k) {
    const int64_t u = m - k;
    const int32_t* idx_in = w.idx[k & 1];
    PairwiseWs pw;
    if (u >= 2) {
      const PairwisePlan p = plan_pairwise(n_eff, u);
      pairwise_ws_bytes(p, w.pw, &pw);
      int rc = run_pairwise(p, pw, cur, ldc, prec, w.Hx, w.Hr, w.S, w.Cov, nullptr, st, stream,
                            k == 0 ? PairwiseStart::kFirst : PairwiseStart::kContinue);
      if (rc) return rc;
      if (k == k_exact) {             // hybrid: the heuristic orders the remaining variables
        rc = run_order(w.S, u, w.osub, margin + k, w.M0, st, stream);
        if (rc) return rc;
        iter_map_kernel<<<(unsigned)ceil_div(u, (int64_t)256), 256, 0, stream>>>(
            w.osub, idx_in, u, order + k);
        VL_LAUNCH_CHECK();
        return VL_OK;
      }
    }
    iter_select_kernel<<<1, kSelThreads, 0, stream>>>(w.S, u, idx_in, k, order, margin, w.pick);
    VL_LAUNCH_CHECK();
    if (u >= 2) {
      float* next = w.D[k & 1];
      // the sums go where the next step's plan keeps them (past this step's means, read here: the
      // sums follow the means, the covariance and the moments)
      PairwiseWs nw;
      pairwise_ws_bytes(plan_pairwise(n_eff, std::max<int64_t>(u - 1, 2)), w.pw, &nw);
      const int splits = colmean_splits(n_eff);
      iter_refine_kernel<<<dim3((unsigned)ceil_div(u - 1, (int64_t)64), (unsigned)splits), 256, 0,
                           stream>>>(cur, ldc, n_eff, u, pw.mu, w.Cov, w.pick, idx_in,
                                     w.idx[(k + 1) & 1], next, m,
                                     ceil_div(n_eff, (int64_t)splits), nw.sums);
      VL_LAUNCH_CHECK();
      cur = next;
      ldc = m;
    }
  }
  return VL_OK;
}

}  // namespace vl
