// Adaptive-lasso pruning of B0 / B_tau (declarations).
#pragma once
#include "common.hpp"

namespace vl {

struct PruneWs {
  int64_t* colmap = nullptr;  // m (p+1) sample offsets of the lag-embedded columns
  double* mu = nullptr;       // their means
  double* C = nullptr;        // m (p+1) square centred cross-products
  double* scratch = nullptr;  // split partials of the covariance
  double* regions = nullptr;  // one LARS state region per variable
};

// Active-set capacity of a path over d columns with at most cap steps (cap 0: no limit).
__host__ __device__ inline int64_t prune_active_cap(int64_t d, int64_t cap) {
  return cap > 0 && cap + 1 < d ? cap + 1 : d;
}
// Doubles of the packed lower-triangular inverse factor of n active columns (blocks of 64 rows,
// padded to whole 64-wide pieces).
__host__ __device__ inline int64_t prune_li_doubles(int64_t n) {
  const int64_t k = ceil_div(n, 64);
  return 2048 * k * (k + 1);
}

// Doubles of the region of a variable with d design columns: the inverse factor, the best knot's
// coefficients, and (designs too long for LDS) ten FP64 vectors and two int32 vectors of d rounded up
// to 64.
__host__ __device__ inline int64_t prune_region_doubles(int64_t d, int64_t cap) {
  return round_up(prune_li_doubles(prune_active_cap(d, cap)) + d + 11 * round_up(d, 64), 32);
}

size_t prune_ws_bytes(int64_t n, int64_t m, int p, int64_t cap, void* base, PruneWs* out);
int run_prune(int64_t n, int64_t m, int p, const PruneWs& w, const float* X, int64_t ldx,
              const int32_t* order, const double* B0, const double* Blag, int64_t cap,
              double* B0_out, double* Blag_out, int32_t* info, int32_t* st, hipStream_t stream);

}  // namespace vl
