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

// MODE 0: out = resid + A W^T + bias (and the optional rounded copy); MODE 1: out = gelu(A W^T + bias).
// TB x TB blocks of 32 x 32 per workgroup.  LN (TB = 1): A is normalised first; its slices stay in registers (K <= 1024).
constexpr int LANE_WAVES = 8, LN_STEPS = 1024 / 16 / LANE_WAVES;
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
      const int c = wave + i * W;
      x[i][0] = x[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (c < nk) {
        x[i][0] = ld4(a32[0] + c * 16);
        x[i][1] = ld4(a32[0] + c * 16 + 4);
        w[i] = *reinterpret_cast<const u32x4*>(wr[0] + c * 16);
      }
    }
    // sum over a row: its pieces in this lane, the other half wavefront's, the other wavefronts'
    auto row_sum = [&](float v, float* buf) {
      v += __shfl_xor(v, 32, 64);
      if (half == 0) buf[wave * 32 + li] = v;
      __syncthreads();
      float t = 0.f;
      for (int k = 0; k < W; ++k) t += buf[k * 32 + li];
      return t;
    };
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < LN_STEPS; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) s += x[i][0][e] + x[i][1][e];
    const float mu = row_sum(s, st) / (float)g.K;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < LN_STEPS; ++i)
      if (wave + i * W < nk) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float c0 = x[i][0][e] - mu, c1 = x[i][1][e] - mu;
          q += c0 * c0 + c1 * c1;
        }
      }
    const float rstd = 1.0f / sqrtf(row_sum(q, st + LANE_WAVES * 32) / (float)g.K + g.eps);
#pragma unroll
    for (int i = 0; i < LN_STEPS; ++i) {
      const int k = (wave + i * W) * 16 + half * 8;
      if (wave + i * W < nk) {
        const f32x4 u0 = (x[i][0] - mu) * rstd * ld4(g.gam + k) + ld4(g.bet + k);
        const f32x4 u1 = (x[i][1] - mu) * rstd * ld4(g.gam + k + 4) + ld4(g.bet + k + 4);
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

// LayerNorm of fp32 rows (D <= 1024): one wavefront per row, statistics in two passes over registers.
__global__ void __launch_bounds__(256) lane_ln_k(const float* __restrict__ x, long long xs, const float* __restrict__ gam,
                                                 const float* __restrict__ bet, float* __restrict__ out, long long os,
                                                 long long rows, int D, float eps) {
  const int lane = threadIdx.x & 63;
  const long long r = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= rows) return;
  float v[16];
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    int d = lane + 64 * i;
    v[i] = d < D ? x[r * xs + d] : 0.f;
    s += v[i];
  }
  const float mu = wave_sum(s) / (float)D;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    int d = lane + 64 * i;
    float c = d < D ? v[i] - mu : 0.f;
    q += c * c;
  }
  const float rstd = 1.0f / sqrtf(wave_sum(q) / (float)D + eps);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    int d = lane + 64 * i;
    if (d < D) out[r * os + d] = (v[i] - mu) * rstd * gam[d] + bet[d];
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
  hipLaunchKernelGGL(lane_ln_k, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, x, xs, gam, bet, out, os, rows, D, eps);
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
  if (N % 64 || K % 64 || n <= 0 || (gam && (K > 1024 || a_bf16 || !gelu)) || (gelu && a_bf16)) return hipErrorInvalidValue;
  LaneGemm g{A, lda, (const bf16*)W, ldw, n, N, K, bias, resid, ldr, out, ldc, (bf16*)copy, ldcopy, gam, bet, eps};
  // 32 x 32 blocks (and the LayerNorm on the way in) up to 524,288 results, 64 x 64 beyond, which read half the operand bytes.
  // (They cross at about 400,000; up to 341 rows of D = 384 all take one form, so that a short slide gives the same bits whole
  // and in chunks: with 64-row chunks on the one and 256 rows on the other the patch embedding's gradients differed by 2.5e-3.)
  // D = 384, us for projection, LayerNorm + fc1, fc2: 200 rows 4.3, 12.5, 11.5 against 8.1, 12.8, 21.7; 332 rows 4.3, 17.4,
  // 11.5 against 8.2, 13.2, 21.6; 2048 rows 7.6, 67, 29 against 8.6, 30, 24.
  const bool small = n * N <= 512 * 1024;
  if (gam && !small) {
    hipLaunchKernelGGL(lane_ln_k, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, (const float*)A, lda, gam, bet, lnout, (long long)K, n, K, eps);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    g.A = lnout; g.lda = K;
  }
  if (gelu) return small ? (gam ? go<1, false, 1, true>(g, s) : go<1, false, 1, false>(g, s)) : go<1, false, 2, false>(g, s);
  if (a_bf16) return small ? go<0, true, 1, false>(g, s) : go<0, true, 2, false>(g, s);
  return small ? go<0, false, 1, false>(g, s) : go<0, false, 2, false>(g, s);
}

}  // namespace sl
