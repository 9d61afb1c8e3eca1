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
// The lane's matrices are a few hundred KB against n rows: what bounds a launch is the serial chain of K steps and their
// trips to L2.  So K is dealt to the (up to eight) wavefronts of a workgroup, each reads its MFMA operands straight from
// global memory with several steps' loads in flight, and the partial blocks are added through LDS.  37 rows of D = 384,
// against 64 x 64 tiles with a 32-wide K loop through LDS: projection 11.1 -> 5.1 us, LayerNorm + fc1 16.3 -> 7.9, fc2 34.4 -> 11.3.
#include "slide_internal.h"

namespace sl {

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

struct LaneGemm {
  const void* A; long long lda;     // fp32 or bf16 [n][K]
  const bf16* W; long long ldw;     // [N][K]
  long long n; int N, K;
  const float* bias;                // [N]
  const float* resid; long long ldr;  // MODE 0
  float* out; long long ldc;
  bf16* copy; long long ldcopy;     // optional bf16 copy of the result rows (MODE 0), may be null
  const float *gam, *bet; float eps;   // LN
};

// eight consecutive k of one row of A as MFMA operands: hi (+ lo for an fp32 A)
struct Frag { bf16x8 hi, lo; };
__device__ __forceinline__ Frag split8(f32x4 a, f32x4 b) {
  Frag f;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    f.hi[e] = (bf16)a[e];
    f.lo[e] = (bf16)(a[e] - (float)f.hi[e]);
    f.hi[4 + e] = (bf16)b[e];
    f.lo[4 + e] = (bf16)(b[e] - (float)f.hi[4 + e]);
  }
  return f;
}

// A LayerNorm's statistics and its output have one order of additions, whichever kernel takes them: a lane holds pieces i of 16
// values starting at (first + 8 i) * 16, half a piece each (x[i][0], x[i][1]: eight neighbours), `row_sum` adds the two halves
// and then the eight lanes' sums in order.
constexpr int LANE_WAVES = 8, LN_STEPS = 1024 / 16 / LANE_WAVES;
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // a caller's vector: any float's address
__device__ __forceinline__ f32x4 ld4u(const float* p) { return *reinterpret_cast<const f32x4u*>(p); }

template <typename F>
__device__ __forceinline__ void ln_stats(const f32x4 (&x)[LN_STEPS][2], int first, int nk, float eps, F row_sum, float& mu, float& rstd) {
  const float D = (float)(nk * 16);
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < LN_STEPS; ++i)   // zeros past the row's end
#pragma unroll
    for (int e = 0; e < 4; ++e) s += x[i][0][e] + x[i][1][e];
  mu = row_sum(s, 0) / D;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < LN_STEPS; ++i)
    if (first + i * LANE_WAVES < nk) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float c0 = x[i][0][e] - mu, c1 = x[i][1][e] - mu;
        q += fmaf(c1, c1, c0 * c0);
      }
    }
  rstd = 1.0f / sqrtf(row_sum(q, 1) / D + eps);
}
__device__ __forceinline__ f32x4 ln_out(f32x4 x, float mu, float rstd, f32x4 gam, f32x4 bet) {
  f32x4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = fmaf((x[e] - mu) * rstd, gam[e], bet[e]);
  return v;
}

// MODE 0: out = resid + A W^T + bias (and the optional rounded copy); MODE 1: out = gelu(A W^T + bias).
// TB x TB blocks of 32 x 32 per workgroup.  LN (TB = 1): A is normalised first; its slices stay in registers (K <= 1024).
template <int MODE, bool A_BF16, int TB, bool LN>
__global__ void __launch_bounds__(64 * LANE_WAVES) lane_gemm_k(LaneGemm g) {
  constexpr int U = TB == 1 ? 6 : 3, NR = TB * TB * 16;   // steps whose loads are issued together, accumulators
  extern __shared__ float red[];   // [W][NR][64] partial blocks
  __shared__ float st[LN ? 2 * LANE_WAVES * 32 : 1];
  const int W = blockDim.x >> 6, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 31, half = lane >> 5;
  const long long m0 = (long long)blockIdx.x * (TB * 32);
  const int n0 = blockIdx.y * (TB * 32), nk = g.K / 16;
  const float* a32[TB];
  const bf16* a16[TB];
  const bf16* wr[TB];
#pragma unroll
  for (int i = 0; i < TB; ++i) {
    long long m = m0 + i * 32 + li;
    if (m > g.n - 1) m = g.n - 1;   // rows past the end re-read the last one and are never stored
    a32[i] = (const float*)g.A + m * g.lda + half * 8;
    a16[i] = (const bf16*)g.A + m * g.lda + half * 8;
    wr[i] = g.W + (long long)(n0 + i * 32 + li) * g.ldw + half * 8;
  }
  f32x16 acc[TB][TB];
#pragma unroll
  for (int i = 0; i < TB; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  auto ld4 = [](const float* p) { return *reinterpret_cast<const f32x4*>(p); };
  if constexpr (LN) {
    static_assert(TB == 1 && !A_BF16, "one block of fp32 rows");
    f32x4 x[LN_STEPS][2];
    u32x4 w[LN_STEPS];
#pragma unroll
    for (int i = 0; i < LN_STEPS; ++i) {
      const int c = wave + i * LANE_WAVES;   // with fewer wavefronts (K < 128) each has one piece
      x[i][0] = x[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (c < nk) {
        x[i][0] = ld4(a32[0] + c * 16);
        x[i][1] = ld4(a32[0] + c * 16 + 4);
        w[i] = *reinterpret_cast<const u32x4*>(wr[0] + c * 16);
      }
    }
    float mu, rstd;
    ln_stats(x, wave, nk, g.eps, [&](float v, int which) {
      float* buf = st + which * (LANE_WAVES * 32);
      v += __shfl_xor(v, 32, 64);
      if (half == 0) buf[wave * 32 + li] = v;
      __syncthreads();
      float t = 0.f;
      for (int k = 0; k < W; ++k) t += buf[k * 32 + li];
      return t;
    }, mu, rstd);
#pragma unroll
    for (int i = 0; i < LN_STEPS; ++i) {
      const int k = (wave + i * LANE_WAVES) * 16 + half * 8;
      if (wave + i * LANE_WAVES < nk) {
        const f32x4 u0 = ln_out(x[i][0], mu, rstd, ld4u(g.gam + k), ld4u(g.bet + k));
        const f32x4 u1 = ln_out(x[i][1], mu, rstd, ld4u(g.gam + k + 4), ld4u(g.bet + k + 4));
        const Frag f = split8(u0, u1);
        const bf16x8 fb = __builtin_bit_cast(bf16x8, w[i]);
        acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.hi, fb, acc[0][0], 0, 0, 0);
        acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.lo, fb, acc[0][0], 0, 0, 0);
      }
    }
  } else {
    for (int c0 = wave; c0 < nk; c0 += U * W) {
      f32x4 x[U][TB][2];
      u32x4 xa[U][TB], w[U][TB];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = c0 + u * W;
        if (c < nk) {
#pragma unroll
          for (int i = 0; i < TB; ++i) {
            if constexpr (A_BF16) {
              xa[u][i] = *reinterpret_cast<const u32x4*>(a16[i] + c * 16);
            } else {
              x[u][i][0] = ld4(a32[i] + c * 16);
              x[u][i][1] = ld4(a32[i] + c * 16 + 4);
            }
            w[u][i] = *reinterpret_cast<const u32x4*>(wr[i] + c * 16);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (c0 + u * W < nk) {
#pragma unroll
          for (int i = 0; i < TB; ++i) {
            Frag f;
            if constexpr (A_BF16) f.hi = __builtin_bit_cast(bf16x8, xa[u][i]);
            else f = split8(x[u][i][0], x[u][i][1]);
#pragma unroll
            for (int j = 0; j < TB; ++j) {
              const bf16x8 fb = __builtin_bit_cast(bf16x8, w[u][j]);
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.hi, fb, acc[i][j], 0, 0, 0);
              if constexpr (!A_BF16) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.lo, fb, acc[i][j], 0, 0, 0);
            }
          }
        }
    }
  }
#pragma unroll
  for (int i = 0; i < TB; ++i)
#pragma unroll
    for (int j = 0; j < TB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) red[(wave * NR + (i * TB + j) * 16 + r) * 64 + lane] = acc[i][j][r];
  __syncthreads();
  // accumulator element r of lane l: row (r / 4) * 8 + (l / 32) * 4 + r % 4, column l % 32 of its block
  for (int k = wave; k < NR; k += W) {
    const int blk = k >> 4, r = k & 15;
    const long long m = m0 + blk / TB * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
    const int col = n0 + blk % TB * 32 + li;
    if (m < g.n) {
      float v = g.bias[col];
      for (int w = 0; w < W; ++w) v += red[(w * NR + k) * 64 + lane];
      if (MODE == 0) {
        v += g.resid[m * g.ldr + col];
        if (g.copy) g.copy[m * g.ldcopy + col] = (bf16)v;
      } else {
        v = gelu_f(v);
      }
      g.out[m * g.ldc + col] = v;
    }
  }
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

// gam: A is normalised first (rows of K, LayerNorm with gam, bet, eps), by a launch of its own into `lnout` on long bags
hipError_t launch_lane_gemm(bool gelu, bool a_bf16, const void* A, long long lda, const void* W, long long ldw, long long n,
                            int N, int K, const float* bias, const float* resid, long long ldr, float* out, long long ldc,
                            void* copy, long long ldcopy, const float* gam, const float* bet, float eps, float* lnout,
                            hipStream_t s) {
  if (N % 64 || K % 64 || n <= 0 || gelu != (gam != nullptr) || (gelu && (K > 1024 || a_bf16))) return hipErrorInvalidValue;
  LaneGemm g{A, lda, (const bf16*)W, ldw, n, N, K, bias, resid, ldr, out, ldc, (bf16*)copy, ldcopy, gam, bet, eps};
  // 32 x 32 blocks (and the LayerNorm on the way in) up to 400,000 results, 64 x 64 beyond, which read half the operand bytes;
  // both give the same bits.  The forward of ViT-S, ms, with the first MLP matrix in the one / in the other form: 200 tiles
  // (307,200 results) 3.838 / 3.846, 275 4.560 / 4.543, 332 5.228 / 5.171; with all three products in the other form: 200 4.21,
  // 340 6.30 against 6.11.  512 tiles: 8.14 with fc1 alone in the other form, 8.22 with none, 8.36 with all.
  const bool small = n * N <= 400000;
  if (gam && !small) {
    hipError_t e = launch_lane_ln((const float*)A, lda, gam, bet, lnout, K, n, K, eps, s);
    if (e != hipSuccess) return e;
    g.A = lnout; g.lda = K;
  }
  if (gelu) return small ? go<1, false, 1, true>(g, s) : go<1, false, 2, false>(g, s);
  if (a_bf16) return small ? go<0, true, 1, false>(g, s) : go<0, true, 2, false>(g, s);
  return small ? go<0, false, 1, false>(g, s) : go<0, false, 2, false>(g, s);
}

}  // namespace sl
