// High-precision lane for the CLS rows of the bf16 path (gfx950).
//
// The slide loss reaches the encoder through one row per tile: the CLS row of the last block (Method: the
// feature matrix is what the aggregator sees).  The aggregator's gate gradients depend on the features only
// through differences between tiles, which are several times smaller than the features themselves, so the
// rounding of that one row is what decides their accuracy: with every CLS row carried in bf16 like the other
// 196 rows of its tile the features are 1e-2 off and the gate gradients 4e-2; with the CLS row's residual
// stream, LayerNorm output, MLP activation and branch sums kept in fp32 they are 1e-3 and 6e-3, while the
// other rows stay on the bf16 kernels.  The lane is n rows out of n * T, so it costs next to nothing.
//
// Per block the lane repeats the row-wise work of the CLS rows (projection + residual, LayerNorm, MLP +
// residual) on an fp32 copy of the CLS stream.  The attention output of the CLS query comes from the main
// path (bf16); after each residual sum the lane writes its value, rounded once, over the CLS row of the main
// path's stream, so the main path's queries, keys, values and saved activations of that row follow the lane.
//   lane_gemm_k : C[n,N] = A[n,K] W[N,K]^T + bias, then + residual or GELU.  W are the bf16 weights of the
//                 step.  An fp32 A is split into two bf16 terms (a = hi + lo up to 2^-17 |a|) and multiplied
//                 in two MFMAs, so the product keeps fp32-grade operands on the bf16 matrix cores; a bf16 A
//                 (rows of the attention output) is exact as it is.  fp32 accumulation, fp32 result.  The LayerNorm
//                 in front of the first MLP matrix is taken on the way in where the bag is short.
//   lane_ln_k   : LayerNorm of fp32 rows, fp32 result.
// Bags of up to 16,384 token rows have no launches for the lane: its products ride in those of the main path that take the same step
// (cls_lane.h, gemm_nt_mid_lane_k, ln_fwd_lane_k).
// The lane's matrices are a few hundred KB against n rows: what bounds a launch is the serial chain of K steps and their
// trips to L2.  So K is dealt to the (up to eight) wavefronts of a workgroup, each reads its MFMA operands straight from
// global memory with several steps' loads in flight, and the partial blocks are added through LDS.  37 rows of D = 384,
// against 64 x 64 tiles with a 32-wide K loop through LDS: projection 11.1 -> 5.1 us, LayerNorm + fc1 16.3 -> 7.9, fc2 34.4 -> 11.3.
#include "cls_lane.h"

namespace sl {

namespace {

template <int MODE, bool A_BF16, int TB, bool LN>
__global__ void __launch_bounds__(64 * LANE_WAVES) lane_gemm_k(LaneGemm g) {
  extern __shared__ float red[];
  __shared__ float st[LN ? 2 * LANE_WAVES * 32 : 1];
  lane_block<MODE, A_BF16, TB, LN>(g, blockIdx.x, blockIdx.y, red, st);
}

// LayerNorm of fp32 rows (D <= 1024, a multiple of 64): 16 lanes per row, two (the halves of a piece) for each wavefront that
// lane_gemm_k deals a row to, so that a bag gives the same bits with the LayerNorm on the way in and in a launch of its own.
__global__ void __launch_bounds__(256) lane_ln_k(const float* __restrict__ x, long long xs, const float* __restrict__ gam,
                                                 const float* __restrict__ bet, float* __restrict__ out, long long os,
                                                 long long rows, int D, float eps) {
  const int lane = threadIdx.x & 63, first = (lane & 15) >> 1, half = lane & 1, nk = D / 16;
  const long long r = (long long)blockIdx.x * 16 + (threadIdx.x >> 4);
  const float* row = x + (r < rows ? r : rows - 1) * xs;   // rows past the end re-read the last one and are never stored
  f32x4 v[LN_STEPS][2];
#pragma unroll
  for (int i = 0; i < LN_STEPS; ++i) {
    const int c = first + i * LANE_WAVES;
    v[i][0] = v[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (c < nk) {
      v[i][0] = ld4u(row + c * 16 + half * 8);
      v[i][1] = ld4u(row + c * 16 + half * 8 + 4);
    }
  }
  float mu, rstd;
  ln_stats(v, first, nk, eps, [&](float s, int) {
    s += __shfl_xor(s, 1, 64);
    float t = 0.f;
#pragma unroll
    for (int k = 0; k < LANE_WAVES; ++k) t += __shfl(s, (lane & ~15) + 2 * k, 64);
    return t;
  }, mu, rstd);
  if (r >= rows) return;
#pragma unroll
  for (int i = 0; i < LN_STEPS; ++i) {
    const int k = (first + i * LANE_WAVES) * 16 + half * 8;
    if (k < D) {
      float* o = out + r * os + k;
      *reinterpret_cast<f32x4u*>(o) = ln_out(v[i][0], mu, rstd, ld4u(gam + k), ld4u(bet + k));
      *reinterpret_cast<f32x4u*>(o + 4) = ln_out(v[i][1], mu, rstd, ld4u(gam + k + 4), ld4u(bet + k + 4));
    }
  }
}

// the CLS stream before the first block: cls + pos[0], the same row for every tile
__global__ void __launch_bounds__(256) lane_init_k(const float* __restrict__ cls, const float* __restrict__ pos,
                                                   float* __restrict__ xc, long long total, int D) {
  long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i < total) { int d = (int)(i % D); xc[i] = cls[d] + pos[d]; }
}

}  // namespace

bool cls_lane_ok(int D, int F) { return D % 64 == 0 && F % 64 == 0 && D <= 1024; }

hipError_t launch_lane_init(const float* cls, const float* pos, float* xc, long long n, int D, hipStream_t s) {
  long long total = n * D;
  hipLaunchKernelGGL(lane_init_k, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, cls, pos, xc, total, D);
  return hipGetLastError();
}

hipError_t launch_lane_ln(const float* x, long long xs, const float* gam, const float* bet, float* out, long long os,
                          long long rows, int D, float eps, hipStream_t s) {
  hipLaunchKernelGGL(lane_ln_k, dim3((unsigned)((rows + 15) / 16)), dim3(256), 0, s, x, xs, gam, bet, out, os, rows, D, eps);
  return hipGetLastError();
}

namespace {

template <int MODE, bool A_BF16, int TB, bool LN>
hipError_t go(const LaneGemm& g, hipStream_t s) {
  const int W = g.K / 16 < LANE_WAVES ? g.K / 16 : LANE_WAVES;
  const size_t lds = (size_t)W * TB * TB * 16 * 64 * 4;
  auto kern = lane_gemm_k<MODE, A_BF16, TB, LN>;
  if (lds > 65536 - 4096) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  const dim3 grid((unsigned)((g.n + TB * 32 - 1) / (TB * 32)), (unsigned)(g.N / (TB * 32)));
  hipLaunchKernelGGL(kern, grid, dim3(64 * W), lds, s, g);
  return hipGetLastError();
}

}  // namespace

// 32 x 32 blocks (and the LayerNorm on the way in) up to 400,000 results, 64 x 64 beyond, which read half the operand bytes;
// both give the same bits.  The forward of ViT-S, ms, with the first MLP matrix in the one / in the other form: 200 tiles
// (307,200 results) 3.838 / 3.846, 275 4.560 / 4.543, 332 5.228 / 5.171; with all three products in the other form: 200 4.21,
// 340 6.30 against 6.11.  512 tiles: 8.14 with fc1 alone in the other form, 8.22 with none, 8.36 with all.
bool lane_small(const LaneGemm& g) { return g.n * g.N <= 400000; }

bool lane_gemm_ok(const LaneGemm& g, bool gelu, bool a_bf16) {
  return g.N % 64 == 0 && g.K % 64 == 0 && g.n > 0 && gelu == (g.gam != nullptr) && !(gelu && (g.K > 1024 || a_bf16));
}

// g.gam: A is normalised first (rows of K, LayerNorm with gam, bet, eps), by a launch of its own into `lnout` on long bags
hipError_t launch_lane_gemm(bool gelu, bool a_bf16, LaneGemm g, float* lnout, hipStream_t s) {
  if (!lane_gemm_ok(g, gelu, a_bf16)) return hipErrorInvalidValue;
  const bool small = lane_small(g);
  if (g.gam && !small) {
    hipError_t e = launch_lane_ln((const float*)g.A, g.lda, g.gam, g.bet, lnout, g.K, g.n, g.K, g.eps, s);
    if (e != hipSuccess) return e;
    g.A = lnout; g.lda = g.K;
  }
  if (gelu) return small ? go<1, false, 1, true>(g, s) : go<1, false, 2, false>(g, s);
  if (a_bf16) return small ? go<0, true, 1, false>(g, s) : go<0, true, 2, false>(g, s);
  return small ? go<0, false, 1, false>(g, s) : go<0, false, 2, false>(g, s);
}

}  // namespace sl
