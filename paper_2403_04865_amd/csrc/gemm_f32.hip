// float32 GEMMs on the bf16 matrix cores, for the float32 path and the float32 contractions of the aggregator.
//
//   NT  C[M,N] = A[M,K] B[N,K]^T + epilogue      TN  C[N1,N2] = sum_m A[m,N1]^T B[m,N2], split over slabs of m
//
// The float32 form of the MFMA does 256 flops a clock and compute unit, a sixteenth of the bf16 rate, and bounded these products
// (105 of the 140 TFLOP/s that it sustains).  So an operand is cut into three bf16 terms of eight bits, whose sum it is exactly, and
// six of the nine products of terms are added in float32: 2.7 times the rate.  What is left out is at most 2^-24 of a product and of either
// sign (terms that are cut off instead of rounded leave out up to 2^-21, always of the product's own sign: sums of positive numbers came out
// 1.35 times as far off as the float32 MFMA's).  Errors against 64 bits, this / the float32 MFMA, normal operands: K = 384 1.1e-7 to 2.9e-7 (by how
// many groups K is dealt to) / 3.5e-7, K = 1536 2.1e-7 to 4.2e-7 / 7.0e-7, sums over M = 12,017 rows 4.5e-7 in 14 slabs / 4.9e-7 in 16; positive
// operands 0.6e-7 to 2.4e-7 / 3.0e-7, 0.8e-7 to 2.2e-7 / 6.0e-7, 0.90e-7 / 1.10e-7; geometric means of the ratio over the encoder's shapes 0.53
// (NT) and 0.85 (TN), positive 0.35 and 0.89.
// Operands are cut once per workgroup, on their way through registers into LDS, the next step's loads in flight meanwhile; the
// vector work of one workgroup (a fifth to a third of the MFMAs' clocks) hides behind the MFMAs of the others, of which three to six fit a
// compute unit with one stage each (two stages and half the workgroups were a quarter slower).  us, before / now: M = 12,017: N = 1536, K = 384
// 122 / 90 (158 TFLOP/s, 0.95 PFLOP/s of bf16), N = 384, K = 1536 123 / 100, weight gradient 1536 x 384 132 / 84.
#include "gemm_epi.h"
#include "lds_dma.h"
#include "split_f32.h"
#include <type_traits>

namespace sl {

namespace {

constexpr int NXCD = 8;
constexpr int BK = SPLIT_BK;   // elements of K (NT) / rows of m (TN) per step

template <int V> using IC = std::integral_constant<int, V>;

// acc[i][j] += 32 x 32 blocks of A (rows oa + 32 i ..) and B (rows ob + 32 j ..), B as the MFMA's first operand
template <int ROWS, int NA, int NB>
__device__ __forceinline__ void mul_step(const bf16* s, int oa, int ob, int half, f32x16 (&acc)[NA][NB]) {
#pragma unroll
  for (int ks = 0; ks < BK / 16; ++ks) {
    Split fa[NA], fb[NB];
#pragma unroll
    for (int i = 0; i < NA; ++i) fa[i] = get_split<ROWS>(s, oa + i * 32, ks * 2 + half);
#pragma unroll
    for (int j = 0; j < NB; ++j) fb[j] = get_split<ROWS>(s, ob + j * 32, ks * 2 + half);
#pragma unroll
    for (int t = 0; t < 6; ++t)
#pragma unroll
      for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j].t[TERM_B[t]], fa[i].t[TERM_A[t]], acc[i][j], 0, 0, 0);
  }
}
// four neighbouring results of row m, columns n .. n + 3
template <int MODE>
__device__ __forceinline__ void epi4(const GemmNT& g, long long m, int n, f32x4 v) {
  const long long mo = MODE == EPI_PATCH ? g.cmap.map32((unsigned)m) : m;
  if constexpr (MODE != EPI_PLAIN && MODE != EPI_DGELU) v += *reinterpret_cast<const f32x4*>(g.bias + n);
  if constexpr (MODE == EPI_BIAS_RESID) v += *reinterpret_cast<const f32x4*>((const float*)g.resid + m * g.ldr + n);
  if constexpr (MODE == EPI_PATCH) v += *reinterpret_cast<const f32x4*>(g.pos + (size_t)(1 + (unsigned)m % (unsigned)g.cmap.g2) * g.N + n);
  if constexpr (MODE == EPI_DGELU) v *= *reinterpret_cast<const f32x4*>((const float*)g.pre + m * g.ldpre + n);
  if constexpr (MODE == EPI_BIAS_GELU) {
    f32x4 d;
#pragma unroll
    for (int e = 0; e < 4; ++e) { float a, b; gelu_both(v[e], &a, &b); v[e] = a; d[e] = b; }
    if (g.out2) *reinterpret_cast<f32x4*>((float*)g.out2 + m * g.ldc2 + n) = d;
  }
  *reinterpret_cast<f32x4*>((float*)g.out + mo * g.ldc + n) = v;
}

// KG groups of four wavefronts deal the K steps among them and add their partial blocks at the end.
template <int BM, int BN, int KG, int MODE>
__global__ void __launch_bounds__(256 * KG, BM + BN == 192 ? 3 : 4) gemm_nt_f32_k(GemmNT g, int MT, int NTL) {
  constexpr int WBM = BM / 64, WBN = BN / 64, ROWS = BM + BN, NU = ROWS / 64;   // NU pieces of eight floats per thread and step
  static_assert(KG == 1 || (WBM == 1 && WBN == 1), "one block per wavefront is added up");
  __shared__ __attribute__((aligned(16))) bf16 stages[KG * 3 * ROWS * BK];
  const int xcd = blockIdx.x % NXCD, slot = blockIdx.x / NXCD;   // the column tiles of a row panel share an XCD's L2
  const int mt = (slot / NTL) * NXCD + xcd;
  if (mt >= MT) return;
  const long long m0 = (long long)mt * BM;
  const int n0 = (slot % NTL) * BN;
  const int tid = threadIdx.x & 255, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);   // this group's steps: grp, grp + KG, ...
  bf16* st = stages + grp * 3 * ROWS * BK;
  const int wm = wave >> 1, wn = wave & 1;
  const int nk = g.K / BK;

  const float* src[NU];   // rows past the end re-read the last one and are never stored
#pragma unroll
  for (int j = 0; j < NU; ++j) {
    const int R = j * 64 + (tid >> 2);
    if (j < BM / 64) {
      long long m = m0 + R;
      if (m > g.M - 1) m = g.M - 1;
      src[j] = (const float*)g.A + g.amap.map32((unsigned)m) * g.lda + (tid & 3) * 8;
    } else {
      long long n = n0 + R - BM;
      if (n > g.N - 1) n = g.N - 1;
      src[j] = (const float*)g.B + n * g.ldb + (tid & 3) * 8;
    }
  }
  f32x4 x[NU][2];
  auto load = [&](int kt) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NU; ++j) {
      x[j][0] = *reinterpret_cast<const f32x4*>(src[j] + kt * BK);
      x[j][1] = *reinterpret_cast<const f32x4*>(src[j] + kt * BK + 4);
    }
  };
  const float up = split_up(grp);
  auto store = [&](bf16* s) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NU; ++j)
      put_split<ROWS>(s, j * 64 + (tid >> 2), tid & 3, split_of(x[j][0], x[j][1], j < BM / 64 ? up : 1.f));
  };
  f32x16 acc[WBM][WBN];
#pragma unroll
  for (int i = 0; i < WBM; ++i)
#pragma unroll
    for (int j = 0; j < WBN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int frow = lane & 31, half = lane >> 5;
  const int oa = wm * (WBM * 32) + frow, ob = BM + wn * (WBN * 32) + frow;
  if (grp < nk) load(grp);
  for (int k0 = 0; k0 < nk; k0 += KG) {   // (the groups meet at the barriers, so they take the same number of turns)
    const int kt = k0 + grp;
    if (k0) step_barrier();   // every wavefront is done with the step before
    if (kt < nk) store(st);
    if (kt + KG < nk) load(kt + KG);
    step_barrier();
    if (kt < nk) mul_step<ROWS>(st, oa, ob, half, acc);
  }
  if (!not_finite(acc)) {
    scale_down(acc, up);
  } else {
#pragma unroll
    for (int i = 0; i < WBM; ++i)
#pragma unroll
      for (int j = 0; j < WBN; ++j) {
        long long m = m0 + (wm * WBM + i) * 32 + frow, n = n0 + (wn * WBN + j) * 32 + frow;
        if (m > g.M - 1) m = g.M - 1;
        if (n > g.N - 1) n = g.N - 1;
        const float *pa = (const float*)g.A + g.amap.map32((unsigned)m) * g.lda + half * 4, *pb = (const float*)g.B + n * g.ldb + half * 4;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
#pragma nounroll
        for (int kt = grp; kt < nk; kt += KG)   // this group's steps and no others: the other groups' blocks stand as they are
#pragma nounroll
          for (int k = kt * BK; k < kt * BK + BK; k += 8) {
            const f32x4 u = *reinterpret_cast<const f32x4*>(pa + k), v = *reinterpret_cast<const f32x4*>(pb + k);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[e], u[e], acc[i][j], 0, 0, 0);
          }
      }
  }

  if constexpr (KG > 1) {   // the groups' partial blocks, in order
    float* red = reinterpret_cast<float*>(stages);   // [KG - 1][16][256]
    static_assert((KG - 1) * 16 * 256 * 4 <= KG * 3 * ROWS * BK * 2, "room");
    __syncthreads();
    if (grp > 0) {
#pragma unroll
      for (int r = 0; r < 16; ++r) red[((grp - 1) * 16 + r) * 256 + tid] = acc[0][0][r];
    }
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int q = 0; q < KG - 1; ++q)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[0][0][r] += red[(q * 16 + r) * 256 + tid];
  }
  // accumulator element r of lane l: row l % 32, column (r / 4) * 8 + (l / 32) * 4 + r % 4 of its block
#pragma unroll
  for (int i = 0; i < WBM; ++i) {
    const long long m = m0 + (wm * WBM + i) * 32 + frow;
    if (m >= g.M) continue;
#pragma unroll
    for (int j = 0; j < WBN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n = n0 + (wn * WBN + j) * 32 + q * 8 + half * 4;
        if (n >= g.N) continue;
        epi4<MODE>(g, m, n, f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]});
      }
  }
}

// NT on few rows: what bounds it there is the serial chain of K steps, so a workgroup has 32 x 32 results and deals K to its
// wavefronts, which read their operands straight from memory, several steps ahead, and add their partial blocks through LDS.
constexpr int SW = 8, SU = 3;   // wavefronts of a workgroup, steps whose loads are issued together
template <int MODE>
__global__ void __launch_bounds__(64 * SW) gemm_nt_f32_few_k(GemmNT g, int NTL) {
  __shared__ float red[SW][16][64];
  const int mt = blockIdx.x / NTL, nt = blockIdx.x % NTL;   // few row tiles: the column tiles are what is dealt to the XCDs
  const int W = blockDim.x >> 6, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 31, half = lane >> 5, nk = g.K / 16;
  const long long m0 = (long long)mt * 32;
  const int n0 = nt * 32;
  const long long m = m0 + li < g.M ? m0 + li : g.M - 1;   // rows past the end re-read the last one and are never stored
  const int n = n0 + li < g.N ? n0 + li : g.N - 1;
  const float* pa = (const float*)g.A + g.amap.map32((unsigned)m) * g.lda;
  const float* pb = (const float*)g.B + (long long)n * g.ldb;
  auto ld4 = [](const float* p) { return *reinterpret_cast<const f32x4*>(p); };
  f32x16 acc[1][1];
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[0][0][r] = 0.f;
  const float up = split_up(wave);
  for (int c0 = wave; c0 < nk; c0 += SU * W) {
    f32x4 x[SU][2], y[SU][2];
#pragma unroll
    for (int u = 0; u < SU; ++u)
      if (c0 + u * W < nk) {
        const int k = (c0 + u * W) * 16 + half * 8;
        x[u][0] = ld4(pa + k); x[u][1] = ld4(pa + k + 4);
        y[u][0] = ld4(pb + k); y[u][1] = ld4(pb + k + 4);
      }
#pragma unroll
    for (int u = 0; u < SU; ++u)
      if (c0 + u * W < nk) {
        const Split fa = split_of(x[u][0], x[u][1], up);
        const Split fb = split_of(y[u][0], y[u][1]);
#pragma unroll
        for (int t = 0; t < 6; ++t) acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb.t[TERM_B[t]], fa.t[TERM_A[t]], acc[0][0], 0, 0, 0);
      }
  }
  if (!not_finite(acc)) {
    scale_down(acc, up);
  } else {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][0][r] = 0.f;
#pragma nounroll
    for (int c = wave; c < nk; c += W)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int k = c * 16 + half * 8 + h * 4;
        const f32x4 u = ld4(pa + k), v = ld4(pb + k);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[e], u[e], acc[0][0], 0, 0, 0);
      }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) red[wave][r][lane] = acc[0][0][r];
  __syncthreads();
  for (int q = wave; q < 4; q += W) {   // columns q * 8 + half * 4 .. + 3 of row li
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    for (int w = 0; w < W; ++w)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += red[w][q * 4 + e][lane];
    const int c = n0 + q * 8 + half * 4;
    if (m0 + li < g.M && c < g.N) epi4<MODE>(g, m0 + li, c, v);
  }
}

template <typename F>
hipError_t by_mode(int epi, F f) {
  switch (epi) {
    case EPI_PLAIN: f(IC<EPI_PLAIN>{}); break;
    case EPI_BIAS: f(IC<EPI_BIAS>{}); break;
    case EPI_BIAS_RESID: f(IC<EPI_BIAS_RESID>{}); break;
    case EPI_BIAS_GELU: f(IC<EPI_BIAS_GELU>{}); break;
    case EPI_DGELU: f(IC<EPI_DGELU>{}); break;
    case EPI_PATCH: f(IC<EPI_PATCH>{}); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
long long tiles_of(long long rows, int cols, int bm, int bn) { return ((rows + bm - 1) / bm) * ((cols + bn - 1) / bn); }

template <int BM, int BN, int KG>
hipError_t go_nt(const GemmNT& g, hipStream_t s) {
  const int MT = (int)((g.M + BM - 1) / BM), NTL = (g.N + BN - 1) / BN;
  const long long wgs = (long long)((MT + NXCD - 1) / NXCD) * NXCD * NTL;
  if (wgs >= (1LL << 31)) return hipErrorInvalidValue;
  return by_mode(g.epi, [&](auto mode) {
    hipLaunchKernelGGL((gemm_nt_f32_k<BM, BN, KG, decltype(mode)::value>), dim3((unsigned)wgs), dim3(256 * KG), 0, s, g, MT, NTL);
  });
}
hipError_t go_nt_few(const GemmNT& g, hipStream_t s) {
  const int W = g.K / 16 < SW ? g.K / 16 : SW;
  return by_mode(g.epi, [&](auto mode) {
    hipLaunchKernelGGL((gemm_nt_f32_few_k<decltype(mode)::value>), dim3((unsigned)tiles_of(g.M, g.N, 32, 32)), dim3(64 * W), 0, s, g, (g.N + 31) / 32);
  });
}

// TN: TB x TB of the result per workgroup.  A thread's pieces of an operand are eight rows of m of one column.
// Rows past the slab's end and columns past the matrix lie outside of the buffers: zeros.  The column sums of A (bias
// gradients) ride along in the registers that A passes through: 16 rows of a step first, then the even and the odd steps.
template <int TB>
__global__ void __launch_bounds__(256, TB == 128 ? 3 : 4) gemm_tn_f32_k(GemmTN g, int per) {
  constexpr int WB = TB / 64, ROWS = 2 * TB, NU = ROWS / 64;   // blocks of a wavefront; NU / 2 pieces of A and of B per thread and step
  __shared__ __attribute__((aligned(16))) bf16 st[3 * ROWS * BK];
  const int i0 = blockIdx.x * TB, j0 = blockIdx.y * TB, slab = blockIdx.z;
  const long long lo = (long long)slab * per, hi = lo + per < g.M ? lo + per : g.M;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wi = wave >> 1, wj = wave & 1;
  const int nk = hi > lo ? (int)((hi - lo + BK - 1) / BK) : 0;

  constexpr int GS = 256 / TB;   // piece j of a thread: rows (tid / TB + j * GS) * 8 .. + 7 of a step, column tid % TB
  const int col = tid % TB, grp = tid / TB;
  const int ao = i0 + col < g.N1 ? (grp * 8 * (int)g.lda + col) * 4 : DMA_ABSENT;
  const int bo = j0 + col < g.N2 ? (grp * 8 * (int)g.ldb + col) * 4 : DMA_ABSENT;
  float x[NU][8];
  auto load = [&](int kt) __attribute__((always_inline)) {
    const long long m = lo + (long long)kt * BK;
    const int rows = hi - m < BK ? (int)(hi - m) : BK;
    const __amdgpu_buffer_rsrc_t ra = dma_rows((const float*)g.A + m * g.lda + i0, rows, (int)g.lda, g.N1 - i0);
    const __amdgpu_buffer_rsrc_t rb = dma_rows((const float*)g.B + m * g.ldb + j0, rows, (int)g.ldb, g.N2 - j0);
#pragma unroll
    for (int j = 0; j < NU / 2; ++j)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        x[j][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ra, ao, (j * GS * 8 + e) * 4 * (int)g.lda, 0));
        x[NU / 2 + j][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, bo, (j * GS * 8 + e) * 4 * (int)g.ldb, 0));
      }
  };
  f32x16 acc[WB][WB];
#pragma unroll
  for (int i = 0; i < WB; ++i)
#pragma unroll
    for (int j = 0; j < WB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  float cs0 = 0.f, cs1 = 0.f;
  const float up = split_up(slab);
  auto store = [&](bf16* s, bool odd) __attribute__((always_inline)) {
    float c = 0.f;
#pragma unroll
    for (int j = 0; j < NU / 2; ++j) {
#pragma unroll
      for (int e = 0; e < 8; ++e) c += x[j][e];
      put_split<ROWS>(s, col, grp + j * GS, split8(x[j], up));
      put_split<ROWS>(s, TB + col, grp + j * GS, split8(x[NU / 2 + j]));
    }
    cs0 += odd ? 0.f : c;
    cs1 += odd ? c : 0.f;
  };
  const int fcol = lane & 31, half = lane >> 5;
  const int oa = wi * (WB * 32) + fcol, ob = TB + wj * (WB * 32) + fcol;
  if (nk > 0) load(0);
  for (int kt = 0; kt < nk; ++kt) {
    if (kt) step_barrier();
    store(st, kt & 1);
    if (kt + 1 < nk) load(kt + 1);
    step_barrier();
    mul_step<ROWS>(st, oa, ob, half, acc);
  }
  if (g.cs_part && blockIdx.y == 0) {
    float* cs = reinterpret_cast<float*>(st);
    __syncthreads();
    cs[tid] = cs0 + cs1;
    __syncthreads();
    if (tid < TB && i0 + tid < g.N1) {
      float c = cs[tid];
#pragma unroll
      for (int q = 1; q < GS; ++q) c += cs[q * TB + tid];
      g.cs_part[(size_t)slab * g.N1 + i0 + tid] = c;
    }
  }
  if (!not_finite(acc)) {
    scale_down(acc, up);
  } else {
#pragma unroll
    for (int i = 0; i < WB; ++i)
#pragma unroll
      for (int j = 0; j < WB; ++j) {
        const int ca = i0 + (wi * WB + i) * 32 + fcol, cb = j0 + (wj * WB + j) * 32 + fcol;
        const float *pa = (const float*)g.A + (ca < g.N1 ? ca : 0), *pb = (const float*)g.B + (cb < g.N2 ? cb : 0);
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
#pragma nounroll
        for (long long m = lo; m < hi; m += 2) {
          const bool ok = m + half < hi;
          const long long row = ok ? m + half : lo;
          const float a = pa[row * g.lda], b = pb[row * g.ldb];
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(ok ? b : 0.f, ok ? a : 0.f, acc[i][j], 0, 0, 0);
        }
      }
  }
  // accumulator element r of lane l: row l % 32, column (r / 4) * 8 + (l / 32) * 4 + r % 4 of its block
  float* P = g.part + (size_t)slab * g.N1 * g.N2;
#pragma unroll
  for (int i = 0; i < WB; ++i) {
    const int row = i0 + (wi * WB + i) * 32 + fcol;
#pragma unroll
    for (int j = 0; j < WB; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = j0 + (wj * WB + j) * 32 + q * 8 + half * 4;
        if (row < g.N1 && c < g.N2)
          *reinterpret_cast<f32x4*>(P + (size_t)row * g.N2 + c) = f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
      }
  }
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace

bool gemm_nt_f32_ok(const GemmNT& g) {
  bool ok = g.K % BK == 0 && g.N % 4 == 0 && g.lda % 4 == 0 && g.ldb % 4 == 0 && g.lda <= DMA_LD && g.ldb <= DMA_LD && g.ldc % 4 == 0 && aligned16(g.A) &&
            aligned16(g.B) && aligned16(g.out) && g.M < (1LL << 31);
  if (g.epi == EPI_BIAS_RESID) ok = ok && g.ldr % 4 == 0 && aligned16(g.resid);
  if (g.epi == EPI_BIAS_GELU) ok = ok && g.ldc2 % 4 == 0 && aligned16(g.out2);
  if (g.epi == EPI_DGELU) ok = ok && g.ldpre % 4 == 0 && aligned16(g.pre);
  if (g.epi == EPI_PATCH) ok = ok && g.cmap.g2 > 0 && aligned16(g.pos);
  if (g.epi != EPI_PLAIN && g.epi != EPI_DGELU) ok = ok && aligned16(g.bias);
  return ok && g.epi != EPI_ROWTAB && g.epi != EPI_TOKEN;
}

// By how many workgroups a problem makes.  us, 32 x 32 / 64 x 64 with K over four, two, one groups / 64 x 128, and the float32 MFMA:
//   32 x 32 up to one per compute unit: 400 rows, N = K = 384 (156) 6.0 / 8.0 8.5 10.2, 9.1; 788 rows (300) 8.9 / 8.1 8.6 10.4, 9.2;
//   four groups up to one 64 x 64 per unit: 2,364 rows, N = 384 (222), K = 384 8.8 9.1 10.9, 9.7; K = 1536 24.5 26.7 36.4, 29.6;
//   two groups up to three, of a longer contraction up to four and a half: 3,152 rows, N = 384 (300), K = 1536 46.4 40.3 45.5, 52.7; 4,728
//   rows (444), K = 384 16.9 14.3 14.8, 16.4; N = 1152 (900) 31.4 24.5 24.3, 28.2; 12,017 rows, N = 384 (1,128), K = 384 29.9 / 29.3, K = 1536 99.9 / 102;
//   64 x 128 from two and a half per unit on: 12,017 rows, N = 384 (564) 29.3 / 31.8, 3,152 rows, N = 1536 (600) 32.6 / 32.4, 6,304 rows, N = 1152 (891)
//   42.6 / 40.7, 12,017 rows, N = 1152 (1,692) 76.1 / 69.8 (128 x 128 is no faster).
hipError_t launch_gemm_nt_f32(const GemmNT& g, hipStream_t s) {
  constexpr int CUS = 256;
  if (tiles_of(g.M, g.N, 32, 32) <= CUS) return go_nt_few(g, s);
  if (tiles_of(g.M, g.N, 64, 128) >= 5 * CUS / 2) return go_nt<64, 128, 1>(g, s);
  const long long t = tiles_of(g.M, g.N, 64, 64);
  if (t <= CUS) return go_nt<64, 64, 4>(g, s);
  if (t <= (g.K >= 768 ? 9 * CUS / 2 : 3 * CUS)) return go_nt<64, 64, 2>(g, s);
  return go_nt<64, 64, 1>(g, s);
}

bool gemm_tn_f32_ok(const GemmTN& g) {
  return g.N1 % 4 == 0 && g.N2 % 4 == 0 && g.lda % 4 == 0 && g.ldb % 4 == 0 && g.lda <= DMA_LD && g.ldb <= DMA_LD && aligned16(g.A) && aligned16(g.B) &&
         g.amap.g2 == 0 && g.bmap.g2 == 0 && g.M < (1LL << 31);
}

// 128 x 128 tiles from 45,000 rows x tiles on.  us, 64 x 64 / 128 x 128: 3,152 rows, 384 x 384 (9 tiles) 13.9 / 14.2, 4,728 18.4 / 16.9; 1,576 rows,
// 1536 x 384 (36) 19.4 / 19.1, 2,364 24.8 / 23.7, 12,017 108.6 / 88.6.
static bool tn_wide(const GemmTN& g) {
  return g.N1 % 128 == 0 && g.N2 % 128 == 0 && g.M * tiles_of(g.N1, g.N2, 128, 128) >= 45000;
}

// Slabs.  128 x 128: two workgroups for every compute unit (three are no faster: 1536 x 384 of 2,364 rows in 14 slabs 23.7 us, in 21 27.3; of
// 12,017 rows 88.6 and 85.8, less than the sum of seven more slabs takes).  64 x 64: nine (two rounds of what fits one at a time), none of less than 128
// rows, since every slab's result is written and read again - except where few tiles would leave units idle, which 32-row slabs may fill.
// Measured with the float32 MFMA: M = 12,017, 192 x 64: 32 slabs 12 us, 8 slabs 39; M = 788, 192 x 64: 32 slabs 3.4 us, 7 slabs 5.6.
// Never fewer than eight of 512 rows: a slab is one chain of float32 additions.
int gemm_tn_f32_slabs(const GemmTN& g, int max_slabs) {
  long long s;
  if (tn_wide(g)) {
    s = 512 / tiles_of(g.N1, g.N2, 128, 128);
  } else {
    const long long tiles = tiles_of(g.N1, g.N2, 64, 64);
    long long by_rows = (g.M + 127) / 128, idle = 512 / tiles;
    s = (2304 + tiles - 1) / tiles;
    if (idle > (g.M + 31) / 32) idle = (g.M + 31) / 32;
    if (by_rows < idle) by_rows = idle;
    if (s > by_rows) s = by_rows;
  }
  long long chain = (g.M + 511) / 512;
  if (chain > 8) chain = 8;
  if (s < chain) s = chain;
  if (s > max_slabs) s = max_slabs;
  return s < 1 ? 1 : (int)s;
}

hipError_t launch_gemm_tn_f32(const GemmTN& g, hipStream_t s) {
  int per = (int)((g.M + g.slabs - 1) / g.slabs);
  per = (per + BK - 1) / BK * BK;
  const int tb = tn_wide(g) ? 128 : 64;
  const dim3 grid((g.N1 + tb - 1) / tb, (g.N2 + tb - 1) / tb, g.slabs);
  if (tb == 128) hipLaunchKernelGGL(gemm_tn_f32_k<128>, grid, dim3(256), 0, s, g, per);
  else hipLaunchKernelGGL(gemm_tn_f32_k<64>, grid, dim3(256), 0, s, g, per);
  return hipGetLastError();
}

}  // namespace sl
