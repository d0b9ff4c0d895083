// One-time precompute of every pairwise entropy statistic (Sec. 4.2 steps 1-2; the first two
// lines of Alg. 1) on gfx950.
//
// Stages (all on the caller's stream):
//   1. column means and the centred covariance of E (FP64 MFMA Gram of the FP32 data);
//   2. standardise (Sec. 3 step 1) and transpose to variable-major Xs (m_pad x n_pad, FP32,
//      zero padded), plus the per-variable moments that give Hx = H(x_i);
//   3. per unordered pair {i,j}: rho = cov/(sd_i sd_j); the Eq. 1 residual of a standardised
//      pair is x_i - rho x_j with variance 1 - rho^2, so the re-standardised residual is
//      u_{i<-j} = (x_i - rho x_j) / sqrt(1 - rho^2); the kernel receives the two scaled
//      coefficients a = c / sqrt(1-rho^2), b = c rho / sqrt(1-rho^2) and forms w = c u;
//   4. the hot kernel: for every pair and sample, both directions w_{i<-j}, w_{j<-i} and their
//      entropy moments (Eq. 2): sum log cosh u and sum u exp(-u^2/2); the micro-tiles holding
//      a near-collinear pair (sqrt(1 - rho^2) < 0.25) are then recomputed by a second kernel
//      that forms their residuals in FP64 from E;
//   5. FP64 combine: Hr = H(nu) - k1 (A - gamma)^2 - k2 B^2 and
//      S[i,j] = (Hx[j] + Hr[i,j]) - (Hx[i] + Hr[j,i]).
#include <algorithm>

#include "gram.hpp"
#include "pairwise.hpp"
#include "pairwise_dev.hpp"
#include "profile.hpp"
#include "sliced.hpp"

namespace vl {

// ------------------------------------------------------------------------------------------
// Kernels (single problem): one body call per block / thread.
// ------------------------------------------------------------------------------------------
// The blocks from nstd on (coef != nullptr) form the pair coefficients and the collinear flags: they
// need the covariance only, as the standardisation does.
__global__ __launch_bounds__(256) void standardize_transpose_kernel(
    const float* __restrict__ E, int64_t lde, int64_t n_eff, int64_t m,
    const double* __restrict__ mu, const double* __restrict__ cov, float* __restrict__ Xs,
    int64_t n_pad, int64_t m_pad, int32_t* st, int64_t nx, int64_t nstd,
    float2* __restrict__ coef, int nt, int32_t* __restrict__ clist) {
  const int64_t b = blockIdx.x;
  if (b < nstd)
    standardize_tile(E, lde, n_eff, m, mu, cov, Xs, n_pad, m_pad, st, (b % nx) * 64,
                     (b / nx) * 64);
  else
    pair_coef_elem(cov, m, m_pad, coef, nt, clist, st, (b - nstd) * 256 + threadIdx.x);
}

// Hx runs in the moments' launch, as its first blocks (one a variable; both read Xs only).  It
// had a launch of its own with the pair coefficients: the exact search at m = 100, n = 5000 6.00
// -> 5.55 ms, the precompute at m = 10, n = 20000 97 -> 91 us, 256 problems 10.97 -> 10.64 ms (a
// launch of m workgroups leaves most of the chip idle for its whole length).  The block after them
// lists the flagged tiles for the collinear kernel.
static inline __host__ __device__ int64_t hx_blocks(int64_t m) { return m / 8 * 8 + 8; }

// Blocks are remapped so that XCD x (block id mod 8) processes a contiguous range of items in
// chunk-major order, i.e. mostly one sample chunk per XCD and its L2.
// TP = float: plain FP32 moment sums; TP = double: compensated sums, FP64 partials.
template <class TP>
__global__ __launch_bounds__(256) void pairwise_moments_kernel(
    const float* __restrict__ Xs, int64_t n_pad, const float2* __restrict__ coef, int64_t m_pad,
    int64_t m, int nt, int64_t tiles, int chunk_len, int64_t items,
    TP* __restrict__ partU, TP* __restrict__ partB, int64_t n_eff, double* __restrict__ Hx,
    double* __restrict__ momx, int32_t* __restrict__ clist) {
  const int64_t nb = gridDim.x - hx_blocks(m);      // a multiple of 8
  const int64_t b = (int64_t)blockIdx.x - hx_blocks(m);
  if (b < 0) {
    if (blockIdx.x < m) hx_block<256>(Xs, n_pad, n_eff, Hx, momx, blockIdx.x);
    else if (blockIdx.x == m && threadIdx.x < 64) list_collinear_tiles(clist, tiles);
    return;
  }
  const int64_t lb = (b & 7) * (nb >> 3) + (b >> 3);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t item = lb * 4 + wave;
  if (item >= items) return;
  if constexpr (std::is_same<TP, double>::value)
    pairwise_moments_item_comp(Xs, n_pad, coef, m_pad, m, nt, tiles, chunk_len, item, partU,
                               partB);
  else
    pairwise_moments_item(Xs, n_pad, coef, m_pad, m, nt, tiles, chunk_len, item, partU, partB);
}

// The (listed tile, chunk) items of the flagged micro-tiles, dealt to the waves one after another
// (flags alone, each wave with a fixed share of all items, gave some waves several and others none:
// m = 400, n = 9998 with 399 near copies 877 us, 750 so); with no flagged tile every wave returns
// after one load.
template <class TP>
__global__ __launch_bounds__(256) void pairwise_collinear_kernel(
    const float* __restrict__ E, int64_t lde, int64_t n_eff, const double* __restrict__ mu,
    const double* __restrict__ cov, int64_t m, int nt, int64_t tiles, int nc, int chunk_len,
    const int32_t* __restrict__ clist, TP* __restrict__ partU, TP* __restrict__ partB) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t total = (int64_t)clist[tiles] * nc, waves = (int64_t)gridDim.x * 4;
  for (int64_t w = (int64_t)blockIdx.x * 4 + wave; w < total; w += waves) {
    const int64_t tile = clist[tiles + 1 + w / nc];
    pairwise_collinear_item(E, lde, n_eff, mu, cov, m, nt, chunk_len, tile, w % nc, partU, partB);
  }
}

// The items' rows, one wave each (see use_rows()); no remap: a handful of items.  A flagged tile's
// item runs as its collinear form instead, on one wave (a launch of its own for those took 3 us).
__global__ __launch_bounds__(256) void pairwise_rows_kernel(
    const float* __restrict__ Xs, int64_t n_pad, const float2* __restrict__ coef, int64_t m_pad,
    int64_t m, int nt, int64_t tiles, int chunk_len, int64_t items, float* __restrict__ partU,
    float* __restrict__ partB, int64_t n_eff, double* __restrict__ Hx, double* __restrict__ momx,
    const float* __restrict__ E, int64_t lde, const double* __restrict__ mu,
    const double* __restrict__ cov, const int32_t* __restrict__ clist) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (blockIdx.x < m) {
    hx_block<256>(Xs, n_pad, n_eff, Hx, momx, blockIdx.x);
    return;
  }
  const int64_t item = (int64_t)blockIdx.x - m;
  if (item >= items) return;
  const int64_t chunk = item / tiles, tile = item - chunk * tiles;
  if (clist[tile]) {
    if (wave == 0)
      pairwise_collinear_item(E, lde, n_eff, mu, cov, m, nt, chunk_len, tile, chunk, partU,
                              partB);
    return;
  }
  pairwise_moments_row(Xs, n_pad, coef, m_pad, m, nt, tiles, chunk_len, item, wave, partU, partB);
}

// blockIdx.x: the upper-triangular blocks of combine_score_block, row by row.
template <class TP>
__global__ __launch_bounds__(kCS * kCS) void combine_score_kernel(
    const TP* __restrict__ partU, const TP* __restrict__ partB, int nc, int64_t m, int64_t n_eff,
    const double* __restrict__ Hx, double* __restrict__ Hr, double* __restrict__ mom,
    double* __restrict__ S, int nb) {
  int bi, bj;
  tile_coords(blockIdx.x, nb, bi, bj);
  combine_score_block(partU, partB, nc, m, n_eff, Hx, Hr, mom, S, bi, bj);
}

// ------------------------------------------------------------------------------------------
// Host side
// ------------------------------------------------------------------------------------------
// Sample chunks: about 16K (tile, chunk) items -- at least 4 chunks, each of at least 512
// samples (4 steps of 2 samples per lane), chunks a multiple of 128.  Measured at one launch
// per fit: m = 400 (n = 10^4) within 1% of the best chunk count, m = 1000 (n = 5 10^4) within
// 0.5%, m = 100 (n = 5000) within 4% (a floor of 2048 samples per chunk was 49% slower there).
PairwisePlan plan_pairwise(int64_t n_eff, int64_t m, bool compensated, bool sliced) {
  PairwisePlan p;
  p.comp = compensated;
  p.sliced = sliced;
  p.m = m;
  p.n_eff = n_eff;
  p.nt = (int)ceil_div(m, kT);
  p.m_pad = (int64_t)p.nt * kT;
  p.tiles = (int64_t)p.nt * (p.nt + 1) / 2;
  const int64_t want = std::max<int64_t>(4, ceil_div(16384, p.tiles));
  const int64_t cap = std::max<int64_t>(1, std::min<int64_t>(512, n_eff / 512));
  p.nc = (int)std::min(want, cap);
  p.chunk_len = (int)round_up(ceil_div(n_eff, p.nc), 128);
  p.n_pad = (int64_t)p.nc * p.chunk_len;
  p.items = p.tiles * p.nc;
  p.blocks = round_up(ceil_div(p.items, 4), 8);
  p.fused = !sliced && cov_sums_fused(m, n_eff);
  return p;
}

// The split partials of the column means and the covariance are dead once the covariance is
// formed, before anything of stages 2-5 is written: the two share one region.
size_t pairwise_ws_bytes(const PairwisePlan& p, void* base, PairwiseWs* out) {
  Carver c(base);
  PairwiseWs w;
  w.mu = c.take<double>(p.m);
  w.cov = c.take<double>(p.m * p.m);
  w.momx = c.take<double>(2 * p.m);
  char* region = base ? static_cast<char*>(base) + c.used : nullptr;
  Carver a(region);                              // stage 1
  w.scratch = a.take<double>(scratch_doubles(p));
  w.sums = w.scratch + (p.fused ? gram_splits_f64(p.m, p.m, p.n_eff) * p.m * p.m : 0);
  if (p.sliced) {
    w.slices = a.take<int8_t>(slice_bytes(p.m, p.n_eff));
    w.ex = a.take<int32_t>(p.m);
  }
  Carver b(region);                              // stages 2-5
  w.Xs = b.take<float>(p.m_pad * p.n_pad);
  w.coef = b.take<float2>(p.m_pad * p.m_pad);
  // FP32 partials, or FP64 ones for the compensated sums (the same region either way)
  const size_t np = (size_t)p.nc * p.m * p.m;
  if (p.comp) {
    w.partU64 = b.take<double>(np);
    w.partB64 = b.take<double>(np);
  } else {
    w.partU = b.take<float>(np);
    w.partB = b.take<float>(np);
  }
  w.clist = b.take<int32_t>(2 * p.tiles + 1);
  if (out) *out = w;
  return c.used + std::max(a.used, b.used);
}

size_t scratch_doubles(const PairwisePlan& p) {
  size_t a = (size_t)colmean_splits(p.n_eff) * p.m;
  size_t b = (size_t)std::max(gram_splits(p.m, p.m, p.n_eff),
                              gram_splits_f64(p.m, p.m, p.n_eff)) * p.m * p.m;
  if (p.sliced) {
    a *= 3;     // column ranges for the slice exponents
    b = std::max(b, (size_t)slice_gram_splits(p.m, p.m, p.n_eff, true) * p.m * p.m);
  }
  // fused: the sums lie past the Gram's own partials, within the scratch where it is larger
  if (p.fused) b = std::max(b, (size_t)gram_splits_f64(p.m, p.m, p.n_eff) * p.m * p.m + a);
  return a > b ? a : b;
}

int standardize_to(const float* E, int64_t lde, int64_t n_eff, int64_t m, const double* mu,
                   const double* cov, float* Xs, int64_t n_pad, int64_t m_pad, int32_t* st,
                   hipStream_t stream, float2* coef, int nt, int32_t* clist) {
  const int64_t nx = ceil_div(n_pad, (int64_t)64), nstd = nx * ceil_div(m_pad, (int64_t)64);
  const int64_t nco = coef ? ceil_div(coef_threads(nt), (int64_t)256) : 0;
  standardize_transpose_kernel<<<(unsigned)(nstd + nco), 256, 0, stream>>>(
      E, lde, n_eff, m, mu, cov, Xs, n_pad, m_pad, st, nx, nstd, coef, nt, clist);
  VL_LAUNCH_CHECK();
  return VL_OK;
}

// Whether a plan's items run as four one-row waves each.  The 1024 SIMDs issue at their limit from
// one wave on, so a plan of x = items / 1024 waves a SIMD takes ceil(x) item times, in rows
// ceil(4 x) / 4 of them, each up to 15% longer for its loads
// (measured: x = 0.01, m = 10, n = 1000 20.0 -> 11.3 us with the launch; 0.44 15.8 -> 10.5; 1.2
// 21.0 -> 15.8; 1.85 and 2.86 even; 16.5 161 -> 171).
static bool use_rows(int64_t items) {
  return 1.15 * (double)ceil_div(4 * items, (int64_t)1024) < 4.0 * (double)ceil_div(items, (int64_t)1024);
}

// Stages 4-5 with FP32 (plain sums) or FP64 (compensated sums) partials.
template <class TP>
static int launch_moments(const PairwisePlan& p, const PairwiseWs& w, const float* E,
                          int64_t lde, const double* cov, double* Hx, double* Hr,
                          double* S, double* mom, TP* partU, TP* partB, hipStream_t stream) {
  const int64_t m = p.m, n_eff = p.n_eff;
  bool rows = false;
  {
    ProfileScope ps("pairwise_moments", stream);
    if constexpr (std::is_same<TP, float>::value) {
      rows = use_rows(p.items);
      if (rows)
        pairwise_rows_kernel<<<(unsigned)(m + p.items), 256, 0, stream>>>(
            w.Xs, p.n_pad, w.coef, p.m_pad, m, p.nt, p.tiles, p.chunk_len, p.items, partU, partB,
            n_eff, Hx, w.momx, E, lde, w.mu, cov, w.clist);
    }
    if (!rows)
      pairwise_moments_kernel<TP><<<(unsigned)(hx_blocks(m) + p.blocks), 256, 0, stream>>>(
          w.Xs, p.n_pad, w.coef, p.m_pad, m, p.nt, p.tiles, p.chunk_len, p.items, partU, partB,
          n_eff, Hx, w.momx, w.clist);
    VL_LAUNCH_CHECK();
  }
  if (!rows) {
    ProfileScope ps("pairwise_collinear", stream);
    const int64_t blocks = std::min<int64_t>(ceil_div(p.items, 4), 256);
    pairwise_collinear_kernel<TP><<<(unsigned)blocks, 256, 0, stream>>>(
        E, lde, n_eff, w.mu, cov, m, p.nt, p.tiles, p.nc, p.chunk_len, w.clist, partU,
        partB);
    VL_LAUNCH_CHECK();
  }
  {
    ProfileScope ps("pairwise_combine", stream);
    const int64_t nb = ceil_div(m, (int64_t)kCS);
    combine_score_kernel<TP><<<(unsigned)(nb * (nb + 1) / 2), kCS * kCS, 0, stream>>>(
        partU, partB, p.nc, m, n_eff, Hx, Hr, mom, S, (int)nb);
    VL_LAUNCH_CHECK();
  }
  return VL_OK;
}

int run_pairwise(const PairwisePlan& p, const PairwiseWs& w, const float* E, int64_t lde,
                 int prec, double* Hx, double* Hr, double* S, double* Cov, double* mom,
                 int32_t* st, hipStream_t stream, PairwiseStart start) {
  const int64_t m = p.m, n_eff = p.n_eff;
  double* cov = Cov ? Cov : w.cov;
  {
    ProfileScope ps("pairwise_cov", stream);
    ColmeanOptions o;
    o.reset = start != PairwiseStart::kContinue;
    o.have_sums = start == PairwiseStart::kContinue;
    if (p.sliced) o.range_exp = w.ex;
    const bool fp32 = (prec & ~VL_PAIRWISE_COMPENSATED) == VL_PREC_FP32;
    const bool fused = p.fused && !fp32;
    o.sums_only = fused;
    int rc = colmeans(E, lde, nullptr, m, n_eff, w.mu, w.sums, st, stream, o);
    if (rc) return rc;
    if (fused) {
      rc = cov_from_sums(E, lde, m, n_eff, w.sums, w.mu, 1.0 / (double)n_eff, cov, w.scratch, st,
                         stream);
      if (rc) return rc;
    } else if (p.sliced) {
      // the covariance from int8 slices of E's centred columns
      rc = slice_columns(E, lde, m, 1, 0, n_eff, w.mu, w.ex, w.slices, stream);
      if (rc) return rc;
      SliceOp D;
      D.D = w.slices;
      D.rows = m;
      D.plane = m * slice_ldk(n_eff);
      D.e = w.ex;
      rc = slice_gram(D, m, D, m, n_eff, 1.0 / (double)n_eff, cov, m, w.scratch, stream, true);
      if (rc) return rc;
    } else {
      // covariance: exact products and FP64 sums (plain FP32 mode: FP32 MFMA throughout)
      rc = gram_tn(E, lde, nullptr, w.mu, m, E, lde, nullptr, w.mu, m, n_eff,
                   fp32 ? GramMode::kFp32 : GramMode::kFp64, 1.0 / (double)n_eff, cov, m,
                   w.scratch, stream, true);
      if (rc) return rc;
    }
  }
  {
    ProfileScope ps("pairwise_prep", stream);
    int rc = standardize_to(E, lde, n_eff, m, w.mu, cov, w.Xs, p.n_pad, p.m_pad, st, stream,
                            w.coef, p.nt, w.clist);
    if (rc) return rc;
  }
  if (p.comp)
    return launch_moments(p, w, E, lde, cov, Hx, Hr, S, mom, w.partU64, w.partB64, stream);
  return launch_moments(p, w, E, lde, cov, Hx, Hr, S, mom, w.partU, w.partB, stream);
}

}  // namespace vl
