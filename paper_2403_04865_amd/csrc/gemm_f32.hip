// float32 GEMMs on the matrix cores (v_mfma_f32_32x32x2_f32: float32 operands, float32 fused multiply-adds), for the
// float32 path and the float32 contractions of the aggregator.  gfx950 has no faster form that keeps 24 bits.
//
//   NT  C[M,N] = A[M,K] B[N,K]^T + epilogue      TN  C[N1,N2] = sum_m A[m,N1]^T B[m,N2], split over slabs of m
//
// What bounds them is the matrix pipe: 256 flops a clock and compute unit, a sixteenth of the bf16 rate, so that a
// 64 x 64 x 32 step lasts 1024 clocks against 16 KB of operands.  Hence small tiles (a bag of a few dozen tiles gives
// several workgroups to every compute unit, and the last wave of workgroups is short), operands straight from global
// memory into LDS one step ahead (lds_dma.h, no registers), one barrier per step, and an epilogue that
// stores from the accumulators.
#include "gemm_epi.h"
#include "lds_dma.h"
#include <type_traits>

namespace sl {

namespace {

constexpr int NXCD = 8;
constexpr int BK = 32;   // floats of K (NT) / rows of m (TN) per step

template <int V> using IC = std::integral_constant<int, V>;

__device__ __forceinline__ void step_barrier() {
  __builtin_amdgcn_s_waitcnt(0x0070);   // this wavefront's loads into LDS have landed, its LDS reads are done
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// NT: rows of 32 floats (128 bytes) in LDS, their 16-byte pieces slot-permuted by the loading lane's choice of address
// (piece c of row R in slot c ^ ((R >> 1) & 7)), so that 16-byte reads of 16 consecutive rows fall on 64 different banks.
// A lane reads four consecutive k of its row at a time and gives one to each of four MFMAs: which two k one MFMA
// multiplies does not matter as long as both operands agree.
template <int BM, int BN, int MODE>
__global__ void __launch_bounds__(256, BM + BN == 256 ? 2 : BM + BN == 192 ? 3 : 4) gemm_nt_f32_k(GemmNT g, int MT, int NTL) {
  constexpr int WBM = BM / 64, WBN = BN / 64;
  constexpr int AG = BM / 32, BG = BN / 32;
  constexpr int STAGE = (BM + BN) * BK;
  constexpr bool HAS_BIAS = MODE != EPI_PLAIN && MODE != EPI_DGELU;
  __shared__ __attribute__((aligned(16))) float st0[STAGE], st1[STAGE];
  const int xcd = blockIdx.x % NXCD, slot = blockIdx.x / NXCD;   // the column tiles of a row panel share an XCD's L2
  const int mt = (slot / NTL) * NXCD + xcd;
  if (mt >= MT) return;
  const long long m0 = (long long)mt * BM;
  const int n0 = (slot % NTL) * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int nk = g.K / BK;

  const int lr = lane >> 3, ls = lane & 7;
  const long long row0 = g.amap.map32((unsigned)m0);
  const __amdgpu_buffer_rsrc_t ra = dma_buffer((const float*)g.A + row0 * g.lda, DMA_MAX);   // (no row past the last one is asked for)
  const __amdgpu_buffer_rsrc_t rb = dma_rows((const float*)g.B + (long long)n0 * g.ldb, g.N - n0 < BN ? g.N - n0 : BN, (int)g.ldb, g.K);
  int ao[AG], bo[BG];
#pragma unroll
  for (int j = 0; j < AG; ++j) {
    const int R = (j * 4 + wave) * 8 + lr;
    long long m = m0 + R;
    if (m > g.M - 1) m = g.M - 1;   // rows past the end re-read the last one and are never stored
    ao[j] = ((int)(g.amap.map32((unsigned)m) - row0) * (int)g.lda + (ls ^ ((R >> 1) & 7)) * 4) * 4;
  }
#pragma unroll
  for (int j = 0; j < BG; ++j) {
    const int R = (j * 4 + wave) * 8 + lr;
    bo[j] = (R * (int)g.ldb + (ls ^ ((R >> 1) & 7)) * 4) * 4;
  }
  auto issue = [&](float* s, int kt) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < AG; ++j) dma16(ra, s + (j * 4 + wave) * 8 * BK, ao[j], kt * BK * 4);
#pragma unroll
    for (int j = 0; j < BG; ++j) dma16(rb, s + BM * BK + (j * 4 + wave) * 8 * BK, bo[j], kt * BK * 4);
  };

  f32x16 acc[WBM][WBN];
#pragma unroll
  for (int i = 0; i < WBM; ++i)
#pragma unroll
    for (int j = 0; j < WBN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int frow = lane & 31, half = lane >> 5, sw = (frow >> 1) & 7;
  const int oa = (wm * (WBM * 32) + frow) * BK, ob = (BM + wn * (WBN * 32) + frow) * BK;
  auto step = [&](const float* s, float* next, int kt) __attribute__((always_inline)) {
    step_barrier();
    if (kt + 1 < nk) issue(next, kt + 1);
#pragma unroll
    for (int ks = 0; ks < BK / 8; ++ks) {
      const int c = ((ks * 2 + half) ^ sw) * 4;
      f32x4 fa[WBM], fb[WBN];
#pragma unroll
      for (int i = 0; i < WBM; ++i) fa[i] = *reinterpret_cast<const f32x4*>(s + oa + i * 32 * BK + c);
#pragma unroll
      for (int j = 0; j < WBN; ++j) fb[j] = *reinterpret_cast<const f32x4*>(s + ob + j * 32 * BK + c);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < WBM; ++i)
#pragma unroll
          for (int j = 0; j < WBN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[j][e], fa[i][e], acc[i][j], 0, 0, 0);
    }
  };
  issue(st0, 0);
  int kt = 0;
  for (; kt + 2 <= nk; kt += 2) {
    step(st0, st1, kt);
    step(st1, st0, kt + 1);
  }
  if (kt < nk) step(st0, st1, kt);

  // accumulator element r of lane l: row l % 32, column (r / 4) * 8 + (l / 32) * 4 + r % 4 of its block
#pragma unroll
  for (int i = 0; i < WBM; ++i) {
    const long long m = m0 + (wm * WBM + i) * 32 + frow;
    if (m >= g.M) continue;
    const long long mo = MODE == EPI_PATCH ? g.cmap.map32((unsigned)m) : m;
    const float* pos = nullptr;
    if constexpr (MODE == EPI_PATCH) pos = g.pos + (size_t)(1 + (unsigned)m % (unsigned)g.cmap.g2) * g.N;
#pragma unroll
    for (int j = 0; j < WBN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n = n0 + (wn * WBN + j) * 32 + q * 8 + half * 4;
        if (n >= g.N) continue;
        f32x4 v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
        if constexpr (HAS_BIAS) v += *reinterpret_cast<const f32x4*>(g.bias + n);
        if constexpr (MODE == EPI_BIAS_RESID) v += *reinterpret_cast<const f32x4*>((const float*)g.resid + m * g.ldr + n);
        if constexpr (MODE == EPI_PATCH) v += *reinterpret_cast<const f32x4*>(pos + n);
        if constexpr (MODE == EPI_DGELU) v *= *reinterpret_cast<const f32x4*>((const float*)g.pre + m * g.ldpre + n);
        if constexpr (MODE == EPI_BIAS_GELU) {
          f32x4 d;
#pragma unroll
          for (int e = 0; e < 4; ++e) { float a, b; gelu_both(v[e], &a, &b); v[e] = a; d[e] = b; }
          if (g.out2) *reinterpret_cast<f32x4*>((float*)g.out2 + m * g.ldc2 + n) = d;
        }
        *reinterpret_cast<f32x4*>((float*)g.out + mo * g.ldc + n) = v;
      }
  }
}

template <int BM, int BN>
hipError_t go_nt(const GemmNT& g, hipStream_t s) {
  const int MT = (int)((g.M + BM - 1) / BM), NTL = (g.N + BN - 1) / BN;
  const long long wgs = (long long)((MT + NXCD - 1) / NXCD) * NXCD * NTL;
  if (wgs >= (1LL << 31)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)wgs), block(256);
  switch (g.epi) {
    case EPI_PLAIN: hipLaunchKernelGGL((gemm_nt_f32_k<BM, BN, EPI_PLAIN>), grid, block, 0, s, g, MT, NTL); break;
    case EPI_BIAS: hipLaunchKernelGGL((gemm_nt_f32_k<BM, BN, EPI_BIAS>), grid, block, 0, s, g, MT, NTL); break;
    case EPI_BIAS_RESID: hipLaunchKernelGGL((gemm_nt_f32_k<BM, BN, EPI_BIAS_RESID>), grid, block, 0, s, g, MT, NTL); break;
    case EPI_BIAS_GELU: hipLaunchKernelGGL((gemm_nt_f32_k<BM, BN, EPI_BIAS_GELU>), grid, block, 0, s, g, MT, NTL); break;
    case EPI_DGELU: hipLaunchKernelGGL((gemm_nt_f32_k<BM, BN, EPI_DGELU>), grid, block, 0, s, g, MT, NTL); break;
    case EPI_PATCH: hipLaunchKernelGGL((gemm_nt_f32_k<BM, BN, EPI_PATCH>), grid, block, 0, s, g, MT, NTL); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// TN: 64 x 64 of the result per workgroup, both operands as [32 rows of m][64 columns] in LDS.  An MFMA operand is one
// float per lane, 32 consecutive columns of one row of m for each half wavefront: a plain read, nothing is transposed.
// Rows past the slab's end and columns past the matrix lie outside of the buffers: zeros.  The column sums of A (bias
// gradients) ride along in the registers that hold A's operands: 16 rows of a step first, then the even and the odd steps.
__global__ void __launch_bounds__(256, 4) gemm_tn_f32_k(GemmTN g, int per) {
  constexpr int STAGE = 2 * BK * 64;
  __shared__ __attribute__((aligned(16))) float st0[STAGE], st1[STAGE];
  const int i0 = blockIdx.x * 64, j0 = blockIdx.y * 64, slab = blockIdx.z;
  const long long lo = (long long)slab * per, hi = lo + per < g.M ? lo + per : g.M;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wi = wave >> 1, wj = wave & 1;
  const int nk = hi > lo ? (int)((hi - lo + BK - 1) / BK) : 0;

  // a load instruction fills 4 rows of 64 floats: instruction j of a wavefront rows (j * 4 + wave) * 4 .. + 3
  const int lr = lane >> 4, lc = (lane & 15) * 4;
  const int ao = i0 + lc < g.N1 ? ((wave * 4 + lr) * (int)g.lda + lc) * 4 : DMA_ABSENT;
  const int bo = j0 + lc < g.N2 ? ((wave * 4 + lr) * (int)g.ldb + lc) * 4 : DMA_ABSENT;
  auto issue = [&](float* s, int kt) __attribute__((always_inline)) {
    const long long m = lo + (long long)kt * BK;
    const int rows = hi - m < BK ? (int)(hi - m) : BK;
    const __amdgpu_buffer_rsrc_t ra = dma_rows((const float*)g.A + m * g.lda + i0, rows, (int)g.lda, g.N1 - i0);
    const __amdgpu_buffer_rsrc_t rb = dma_rows((const float*)g.B + m * g.ldb + j0, rows, (int)g.ldb, g.N2 - j0);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int R = (j * 4 + wave) * 4;
      dma16(ra, s + R * 64, ao, j * 64 * (int)g.lda);
      dma16(rb, s + BK * 64 + R * 64, bo, j * 64 * (int)g.ldb);
    }
  };
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  float cs0 = 0.f, cs1 = 0.f;
  const int fcol = lane & 31, half = lane >> 5;
  auto step = [&](const float* s, float* next, int kt, float& cs) __attribute__((always_inline)) {
    step_barrier();
    if (kt + 1 < nk) issue(next, kt + 1);
    float c16 = 0.f;
    const float* sa = s + half * 64 + wi * 32 + fcol;
    const float* sb = s + BK * 64 + half * 64 + wj * 32 + fcol;
#pragma unroll
    for (int k = 0; k < BK; k += 2) {
      const float a = sa[k * 64], b = sb[k * 64];
      c16 += a;
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
    }
    cs += c16;
  };
  if (nk > 0) issue(st0, 0);
  int kt = 0;
  for (; kt + 2 <= nk; kt += 2) {
    step(st0, st1, kt, cs0);
    step(st1, st0, kt + 1, cs1);
  }
  if (kt < nk) step(st0, st1, kt, cs0);
  if (g.cs_part && blockIdx.y == 0 && wj == 0) {
    float cs = cs0 + cs1;
    cs += __shfl_xor(cs, 32, 64);
    const int i = i0 + wi * 32 + fcol;
    if (half == 0 && i < g.N1) g.cs_part[(size_t)slab * g.N1 + i] = cs;
  }
  float* P = g.part + (size_t)slab * g.N1 * g.N2;
  const int c = j0 + wj * 32 + fcol;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = i0 + wi * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
    if (c < g.N2 && row < g.N1) P[(size_t)row * g.N2 + c] = acc[r];
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

// 64 x 64 tiles at every size: measured against 64 x 128 and 128 x 128 tiles of the same kernel over M = 68 .. 12,017 (all the
// encoder's shapes) they are the fastest throughout.  M = 12,017: N = 1536, K = 384 143 us (99 TFLOP/s; the pipe alone sustains
// 140), 148 and 159 with the larger tiles, 474 with the vector kernel; N = 384, K = 1536 150 us, 175, 211, 445.
hipError_t launch_gemm_nt_f32(const GemmNT& g, hipStream_t s) { return go_nt<64, 64>(g, s); }

bool gemm_tn_f32_ok(const GemmTN& g) {
  return g.N1 % 4 == 0 && g.N2 % 4 == 0 && g.lda % 4 == 0 && g.ldb % 4 == 0 && g.lda <= DMA_LD && g.ldb <= DMA_LD && aligned16(g.A) && aligned16(g.B) &&
         g.amap.g2 == 0 && g.bmap.g2 == 0 && g.M < (1LL << 31);
}

// Slabs: nine workgroups for every compute unit (two rounds of what fits one at a time), none of less than 128 rows, since every
// slab's result is written and read again - except where few tiles would leave units idle, which 32-row slabs may fill.
// Measured: M = 12,017, 1536 x 384: 16 slabs 151 us, 9 slabs 165, 4 slabs 191 (258 .. 274 with the vector kernel); 192 x 64: 32
// slabs 12 us, 8 slabs 39; M = 788, 192 x 64: 32 slabs 3.4 us, 7 slabs 5.6.
// Never fewer than eight of 512 rows: a slab is one chain of float32 additions, two rows each.
int gemm_tn_f32_slabs(const GemmTN& g, int max_slabs) {
  const long long tiles = (long long)((g.N1 + 63) / 64) * ((g.N2 + 63) / 64);
  long long s = (2304 + tiles - 1) / tiles, by_rows = (g.M + 127) / 128, idle = 512 / tiles;
  if (idle > (g.M + 31) / 32) idle = (g.M + 31) / 32;
  if (by_rows < idle) by_rows = idle;
  if (s > by_rows) s = by_rows;
  long long chain = (g.M + 511) / 512;
  if (chain > 8) chain = 8;
  if (s < chain) s = chain;
  if (s > max_slabs) s = max_slabs;
  return s < 1 ? 1 : (int)s;
}

hipError_t launch_gemm_tn_f32(const GemmTN& g, hipStream_t s) {
  int per = (int)((g.M + g.slabs - 1) / g.slabs);
  per = (per + BK - 1) / BK * BK;
  const dim3 grid((g.N1 + 63) / 64, (g.N2 + 63) / 64, g.slabs);
  hipLaunchKernelGGL(gemm_tn_f32_k, grid, dim3(256), 0, s, g, per);
  return hipGetLastError();
}

}  // namespace sl
