// The CLS lane's products (cls_lane.hip) as parts of a workgroup, for the lane's own launches and for those of the short bags that carry a
// piece of the lane beside their own work.
#pragma once
#include "slide_internal.h"

namespace sl {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

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

// K is dealt to this many wavefronts (whose partial sums are added in order), in whatever number of wavefronts that takes
__device__ __forceinline__ int lane_parts(int nk) { return nk < LANE_WAVES ? nk : LANE_WAVES; }

template <int MODE>
__device__ __forceinline__ void lane_store(const LaneGemm& g, long long m, int col, float v) {
  if (MODE == 0) {
    v += g.resid[m * g.ldr + col];
    if (g.copy) g.copy[m * g.ldcopy + col] = (bf16)v;
  } else {
    v = gelu_f(v);
  }
  g.out[m * g.ldc + col] = v;
}

// MODE 0: out = resid + A W^T + bias (and the optional rounded copy); MODE 1: out = gelu(A W^T + bias).
// TB x TB blocks of 32 x 32 per workgroup.  LN (TB = 1): A is normalised first; its slices stay in registers (K <= 1024).
// Workgroup (bx, by) of such a product, in a workgroup of LANE_WAVES wavefronts or of as many as K has pieces of 16.
// red: [wavefronts][TB TB 16][64] partial blocks; st: 2 LANE_WAVES 32 floats (LN)
template <int MODE, bool A_BF16, int TB, bool LN>
__device__ __forceinline__ void lane_block(const LaneGemm& g, int bx, int by, float* red, float* st) {
  constexpr int U = TB == 1 ? 6 : 3, NR = TB * TB * 16;   // steps whose loads are issued together, accumulators
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 31, half = lane >> 5;
  const long long m0 = (long long)bx * (TB * 32);
  const int n0 = by * (TB * 32), nk = g.K / 16, W = lane_parts(nk), waves = blockDim.x >> 6;
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
    for (int c0 = wave < W ? wave : nk; c0 < nk; c0 += U * W) {
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
  for (int k = wave; k < NR; k += waves) {
    const int blk = k >> 4, r = k & 15;
    const long long m = m0 + blk / TB * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
    const int col = n0 + blk % TB * 32 + li;
    if (m < g.n) {
      float v = g.bias[col];
      for (int w = 0; w < W; ++w) v += red[(w * NR + k) * 64 + lane];
      lane_store<MODE>(g, m, col, v);
    }
  }
}

// A 32 x 32 block of a MODE 0 product in a workgroup of four wavefronts, each with two of the eight parts of K: the same sums in the
// same order.  lo, hi: [4][16][64] floats each
template <bool A_BF16>
__device__ __forceinline__ void lane_block4(const LaneGemm& g, int bx, int by, float* lo, float* hi) {
  constexpr int U = 3;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 31, half = lane >> 5;
  const long long m0 = (long long)bx * 32;
  const int n0 = by * 32, nk = g.K / 16, W = lane_parts(nk);
  long long m = m0 + li;
  if (m > g.n - 1) m = g.n - 1;   // rows past the end re-read the last one and are never stored
  const float* a32 = (const float*)g.A + m * g.lda + half * 8;
  const bf16* a16 = (const bf16*)g.A + m * g.lda + half * 8;
  const bf16* wr = g.W + (long long)(n0 + li) * g.ldw + half * 8;
  f32x16 acc[2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
  for (int t0 = 0; t0 * W + wave < nk; t0 += U) {
    f32x4 x[U][2][2];
    u32x4 xa[U][2], w[U][2];
    auto piece = [&](int u, int i) __attribute__((always_inline)) { return wave + 4 * i < W ? (t0 + u) * W + wave + 4 * i : nk; };
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (const int c = piece(u, i); c < nk) {
          if constexpr (A_BF16) {
            xa[u][i] = *reinterpret_cast<const u32x4*>(a16 + c * 16);
          } else {
            x[u][i][0] = *reinterpret_cast<const f32x4*>(a32 + c * 16);
            x[u][i][1] = *reinterpret_cast<const f32x4*>(a32 + c * 16 + 4);
          }
          w[u][i] = *reinterpret_cast<const u32x4*>(wr + c * 16);
        }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (piece(u, i) < nk) {
          Frag f;
          if constexpr (A_BF16) f.hi = __builtin_bit_cast(bf16x8, xa[u][i]);
          else f = split8(x[u][i][0], x[u][i][1]);
          const bf16x8 fb = __builtin_bit_cast(bf16x8, w[u][i]);
          acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.hi, fb, acc[i], 0, 0, 0);
          if constexpr (!A_BF16) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.lo, fb, acc[i], 0, 0, 0);
        }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    lo[(wave * 16 + r) * 64 + lane] = acc[0][r];
    hi[(wave * 16 + r) * 64 + lane] = acc[1][r];
  }
  __syncthreads();
  for (int k = wave; k < 16; k += 4) {
    const long long row = m0 + (k >> 2) * 8 + half * 4 + (k & 3);
    const int col = n0 + li;
    if (row < g.n) {
      float v = g.bias[col];
      for (int q = 0; q < W; ++q) v += (q < 4 ? lo : hi)[((q & 3) * 16 + k) * 64 + lane];
      lane_store<0>(g, row, col, v);
    }
  }
}

}  // namespace sl
