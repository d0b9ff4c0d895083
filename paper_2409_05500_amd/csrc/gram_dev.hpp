// Block-wide centred Gram tiles on gfx950 MFMA, shared by the single-problem kernels (split-K
// partials) and the batched kernels (one tile of one problem per block).
#pragma once
#include "common.hpp"

namespace vl {

// ------------------------------------------------------------------------------------------
// Centred TN Gram tile:  out[i * ldo + j] = scale * sum_{kb <= t < ke} (A(t,i) - muA[i])
// (with `mirror`, also out[j * ldo + i]: the other triangle of a symmetric result)
// (B(t,j) - muB[j]) for i in [i0, i0 + 64), j in [j0, j0 + 64), with A(t,i) = A[mapA[i] +
// t * lda].  Block tile 64 x 64 (4 waves of 32 x 32, one v_mfma_f32_32x32x2f32 accumulator
// each), 32 samples per LDS stage.  kFlush > 0 adds the FP32 accumulator into FP64 registers
// every kFlush stages (FP32-accurate result); kFlush == 0 keeps a plain FP32 accumulator.
// ------------------------------------------------------------------------------------------
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kGT = 64;    // tile side
constexpr int kGK = 32;    // samples per stage
constexpr int kGLd = 65;   // LDS row stride (floats): odd to keep the two half-waves apart

template <int kFlush>
__device__ inline void gram_tile_f32(
    const float* __restrict__ A, int64_t lda, const int64_t* __restrict__ mapA,
    const double* __restrict__ muA, int64_t M, const float* __restrict__ B, int64_t ldb,
    const int64_t* __restrict__ mapB, const double* __restrict__ muB, int64_t N, int64_t i0,
    int64_t j0, int64_t kb, int64_t ke, double* __restrict__ out, int64_t ldo, double scale,
    bool mirror = false) {
  __shared__ float As[kGK * kGLd];
  __shared__ float Bs[kGK * kGLd];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  // loader: column cc, rows rg + 4 r
  const int cc = tid & 63, rg = tid >> 6;
  const int64_t ia = i0 + cc, jb = j0 + cc;
  const bool va = ia < M, vb = jb < N;
  const float* pa = A + (va ? (mapA ? mapA[ia] : ia) : 0);
  const float* pb = B + (vb ? (mapB ? mapB[jb] : jb) : 0);
  const float ma = va ? (float)muA[ia] : 0.f;
  const float mb = vb ? (float)muB[jb] : 0.f;
  // Centring with the float-rounded mean leaves an offset d ~ 1e-8 |mu|; it changes the Gram
  // by K d_a d_b only, since the centred columns sum to zero.

  const int wi = wave >> 1, wj = wave & 1;
  f32x16 acc = {};
  double acc64[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) acc64[r] = 0.0;

  // register prefetch of the next stage overlaps its loads with this stage's MFMAs: the raw
  // values are held, and centred and masked when they are stored to LDS (an operation on a
  // loaded value right after its load would wait for it before the MFMAs)
  float ra[kGK / 4], rb[kGK / 4];
  auto load = [&](int64_t k0) {
#pragma unroll
    for (int r = 0; r < kGK / 4; ++r) {
      const int64_t t = k0 + rg + 4 * r;
      const int64_t tc = t < ke ? t : ke - 1;     // clamped, in bounds; padding masked below
      ra[r] = pa[tc * lda];
      rb[r] = pb[tc * ldb];
    }
  };
  load(kb);
  int stage = 0;
  for (int64_t k0 = kb; k0 < ke; k0 += kGK, ++stage) {
#pragma unroll
    for (int r = 0; r < kGK / 4; ++r) {
      const bool in = k0 + rg + 4 * r < ke;
      As[(rg + 4 * r) * kGLd + cc] = mask_f32(ra[r] - ma, va && in);
      Bs[(rg + 4 * r) * kGLd + cc] = mask_f32(rb[r] - mb, vb && in);
    }
    __syncthreads();
    if (k0 + kGK < ke) load(k0 + kGK);
#pragma unroll
    for (int kk = 0; kk < kGK; kk += 2) {
      const float a = As[(kk + (lane >> 5)) * kGLd + wi * 32 + (lane & 31)];
      const float b = Bs[(kk + (lane >> 5)) * kGLd + wj * 32 + (lane & 31)];
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
    }
    __syncthreads();
    if (kFlush > 0 && (stage % kFlush) == kFlush - 1) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        acc64[r] += (double)acc[r];
        acc[r] = 0.f;
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) acc64[r] += (double)acc[r];

  // D layout of 32x32x2: lane l, reg r -> row 8*(r/4) + 4*(l/32) + r%4, column l%32
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int64_t i = i0 + wi * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    const int64_t j = j0 + wj * 32 + (lane & 31);
    if (i < M && j < N) {
      out[i * ldo + j] = scale * acc64[r];
      if (mirror) out[j * ldo + i] = scale * acc64[r];
    }
  }
}

// ------------------------------------------------------------------------------------------
// BF16 variant (the low-precision Gram that iterative refinement repairs): the centred FP32
// values staged in LDS are rounded to BF16 (nearest, ties to even) when read; the products of
// two BF16 values are exact in FP32; v_mfma_f32_32x32x8bf16_1k (lane l holds A[l % 32][4 (l /
// 32) + 0..3] and B[4 (l / 32) + 0..3][l % 32]; the output layout of the FP32 32x32 MFMA); FP32
// partial sums added into FP64 every 4 stages (128 samples).
// ------------------------------------------------------------------------------------------
typedef short s16x4 __attribute__((ext_vector_type(4)));

__device__ inline short to_bf16(float x) {
  uint32_t u = __float_as_uint(x);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (short)(u >> 16);
}

__device__ inline void gram_tile_bf16(
    const float* __restrict__ A, int64_t lda, const int64_t* __restrict__ mapA,
    const double* __restrict__ muA, int64_t M, const float* __restrict__ B, int64_t ldb,
    const int64_t* __restrict__ mapB, const double* __restrict__ muB, int64_t N, int64_t i0,
    int64_t j0, int64_t kb, int64_t ke, double* __restrict__ out, int64_t ldo, double scale) {
  __shared__ float As[kGK * kGLd];
  __shared__ float Bs[kGK * kGLd];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int cc = tid & 63, rg = tid >> 6;
  const int64_t ia = i0 + cc, jb = j0 + cc;
  const bool va = ia < M, vb = jb < N;
  const float* pa = A + (va ? (mapA ? mapA[ia] : ia) : 0);
  const float* pb = B + (vb ? (mapB ? mapB[jb] : jb) : 0);
  const float ma = va ? (float)muA[ia] : 0.f;
  const float mb = vb ? (float)muB[jb] : 0.f;
  const int wi = wave >> 1, wj = wave & 1;
  f32x16 acc = {};
  double acc64[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) acc64[r] = 0.0;
  float ra[kGK / 4], rb[kGK / 4];
  auto load = [&](int64_t k0) {
#pragma unroll
    for (int r = 0; r < kGK / 4; ++r) {
      const int64_t t = k0 + rg + 4 * r;
      const bool in = t < ke;
      const int64_t tc = in ? t : ke - 1;         // clamped, in bounds; padding masked below
      ra[r] = mask_f32(pa[tc * lda] - ma, va && in);
      rb[r] = mask_f32(pb[tc * ldb] - mb, vb && in);
    }
  };
  load(kb);
  int stage = 0;
  for (int64_t k0 = kb; k0 < ke; k0 += kGK, ++stage) {
#pragma unroll
    for (int r = 0; r < kGK / 4; ++r) {
      As[(rg + 4 * r) * kGLd + cc] = ra[r];
      Bs[(rg + 4 * r) * kGLd + cc] = rb[r];
    }
    __syncthreads();
    if (k0 + kGK < ke) load(k0 + kGK);
#pragma unroll
    for (int kk = 0; kk < kGK; kk += 8) {
      s16x4 a, b;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = kk + 4 * (lane >> 5) + q;
        a[q] = to_bf16(As[k * kGLd + wi * 32 + (lane & 31)]);
        b[q] = to_bf16(Bs[k * kGLd + wj * 32 + (lane & 31)]);
      }
      acc = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(a, b, acc, 0, 0, 0);
    }
    __syncthreads();
    if ((stage & 3) == 3) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        acc64[r] += (double)acc[r];
        acc[r] = 0.f;
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    acc64[r] += (double)acc[r];
    const int64_t i = i0 + wi * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    const int64_t j = j0 + wj * 32 + (lane & 31);
    if (i < M && j < N) out[i * ldo + j] = scale * acc64[r];
  }
}

// ------------------------------------------------------------------------------------------
// FP64 variant: a 64 x 64 tile by v_mfma_f64_16x16x4f64.  FP32 inputs are widened and centred in
// FP64, so every product is exact and the sum is FP64 throughout.
// What bounds it: the FP64 matrix rate, ~60 TFLOP/s sustained, to which every vector operation
// beside a product adds its own issue time (the FP64 matrix and vector units are one).  Hence
// each of the four waves forms the whole tile over a quarter of the samples, straight from
// global memory in the operands' own layout (four rows of 16 consecutive values a load): 16
// products for 8 loads, 8 conversions and 8 subtractions, no LDS and no barrier in the loop, the
// same work for every wave whatever part of an edge tile is live, and a chain a quarter as long.
// A step's values are loaded again for the next group as soon as they are converted (16 samples,
// 64 products, ahead), without a condition: behind a branch the compiler cannot count the
// loads and waits for all.  The quarters are added through LDS in wave
// order at the end.  Two waves per SIMD (128 accumulator registers).
// Measured against the former form (raw values staged in LDS, widened, centred and masked at each
// use): 1000 x 1000 over 49999 samples (lower tiles) 1.43 -> 0.93 ms (60 TFLOP/s of the tiles),
// 400 x 2000 over 9996 0.46 -> 0.35 ms, 10 x 10 over 999 22.6 -> 6.3 us; both Grams of the 256
// uneven problems (m 20-200, n 500-8000) 2.67 -> 1.77 ms, of 181 windows of 50 x 2000 0.38 -> 0.23.
// diag: a tile on the diagonal of a symmetric product forms its lower 16 x 16 blocks only, 10 of
// 16, and writes both halves (the two cases again: 1.77 -> 1.60 ms, 0.23 -> 0.21).
// ------------------------------------------------------------------------------------------
typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kGS64 = 16;    // samples per group of loads

__device__ __forceinline__ void gram_tile_f64(
    const float* __restrict__ A, int64_t lda, const int64_t* __restrict__ mapA,
    const double* __restrict__ muA, int64_t M, const float* __restrict__ B, int64_t ldb,
    const int64_t* __restrict__ mapB, const double* __restrict__ muB, int64_t N, int64_t i0,
    int64_t j0, int64_t kb, int64_t ke, double* __restrict__ out, int64_t ldo, double scale,
    bool mirror = false, bool diag = false) {
  __shared__ double part[4][8][4][64];
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // live 16-wide blocks of the tile; columns past the edge read column 0 (their products land in
  // rows and columns that are not written)
  const int na = (int)(M - i0 < 64 ? (M - i0 + 15) / 16 : 4);
  const int nb = (int)(N - j0 < 64 ? (N - j0 + 15) / 16 : 4);
  const float *pa[4], *pb[4];
  double ma[4], mb[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t ia = i0 + 16 * q + li, jb = j0 + 16 * q + li;
    pa[q] = A + (ia < M ? (mapA ? mapA[ia] : ia) : 0);
    pb[q] = B + (jb < N ? (mapB ? mapB[jb] : jb) : 0);
    ma[q] = ia < M ? muA[ia] : 0.0;
    mb[q] = jb < N ? muB[jb] : 0.0;
  }
  f64x4 acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
  // this wave's samples: whole groups, but for the last wave that has any
  const int64_t K = ke - kb, len = K > 0 ? round_up(ceil_div(K, (int64_t)4), kGS64) : 0;
  const int64_t k0w = kb + wave * len, k1w = k0w + len < ke ? k0w + len : ke;
  const int64_t ng = k1w > k0w ? (k1w - k0w) / kGS64 : 0;
  constexpr int kSteps = kGS64 / 4;
  float xa[kSteps][4], xb[kSteps][4];
  auto products = [&](const double (&av)[4], const double (&bv)[4]) {
#pragma unroll
    for (int a = 0; a < 4; ++a)
      if (a < na) {
        const int nba = diag && a + 1 < nb ? a + 1 : nb;
#pragma unroll
        for (int b = 0; b < 4; ++b)
          if (b < nba)
            acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc[a][b], 0, 0, 0);
      }
  };
  if (ng > 0) {
    const float *qa[4], *qb[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      qa[q] = pa[q] + lk * lda;
      qb[q] = pb[q] + lk * ldb;
    }
    auto load = [&](int64_t t, int s) {              // t wave-uniform
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        xa[s][q] = qa[q][t * lda];
        xb[s][q] = qb[q][t * ldb];
      }
    };
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
      load(k0w + 4 * s, s);
      __builtin_amdgcn_sched_barrier(0);
    }
    const int64_t last = k0w + (ng - 1) * kGS64;
    for (int64_t k0 = k0w; k0 <= last; k0 += kGS64) {
      const int64_t kn = k0 < last ? k0 + kGS64 : last;    // (past the end: the last group again)
#pragma unroll
      for (int s = 0; s < kSteps; ++s) {
        double av[4], bv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          av[q] = (double)xa[s][q] - ma[q];
          bv[q] = (double)xb[s][q] - mb[q];
          asm volatile("" : "+v"(av[q]), "+v"(bv[q]));   // formed here, not at each product
        }
        load(kn + 4 * s, s);
        __builtin_amdgcn_sched_barrier(0);               // (loads stay in this order)
        products(av, bv);
      }
    }
  }
  for (int64_t t0 = k0w + ng * kGS64; t0 < k1w; t0 += 4) {   // the rest: clamped and masked
    const int64_t t = t0 + lk, tc = t < k1w ? t : k1w - 1;
    double av[4], bv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      xa[0][q] = pa[q][tc * lda];
      xb[0][q] = pb[q][tc * ldb];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      av[q] = t < k1w ? (double)xa[0][q] - ma[q] : 0.0;
      bv[q] = t < k1w ? (double)xb[0][q] - mb[q] : 0.0;
    }
    products(av, bv);
  }
  // D layout of 16x16x4 f64: lane l, reg r -> row l/16 + 4 r, column l%16.  Two block rows at a
  // time: every wave leaves its sums in LDS, then adds up and writes two of the eight blocks.
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (2 * h >= na) break;
    if (h > 0) __syncthreads();
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) part[wave][4 * a + b][r][lane] = acc[2 * h + a][b][r];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int blk = 2 * wave + u, a = 2 * h + (blk >> 2), b = blk & 3;
      if (a >= na || b >= nb || (diag && b > a)) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double v = ((part[0][blk][r][lane] + part[1][blk][r][lane]) +
                          part[2][blk][r][lane]) + part[3][blk][r][lane];
        const int64_t i = i0 + a * 16 + lk + 4 * r, j = j0 + b * 16 + li;
        if (i < M && j < N) {
          out[i * ldo + j] = scale * v;
          if (mirror || (diag && a != b)) out[j * ldo + i] = scale * v;
        }
      }
    }
  }
}

}  // namespace vl
