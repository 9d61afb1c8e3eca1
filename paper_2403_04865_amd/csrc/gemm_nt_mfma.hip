// bf16 MFMA "NT" GEMM for gfx950, small and medium M: C[M,N] = A[M,K] * B[N,K]^T (+ fused epilogue), fp32 accumulate.
//
// Every activation-side GEMM of the encoder has this form (forward GEMMs use W [out][in]; input-gradient GEMMs use the
// pre-transposed copy W^T, so both operands are always K-contiguous).  The large-M kernels (gemm_nt_big.hip,
// gemm_nt_gelu.hip) take a whole slide; this one takes the problems whose 256 x 192 tiles would leave most compute
// units idle: bags of a few tiles up to a few hundred, the CLS rows of the last block, narrow encoders.
//
// What bounds such a problem is latency, not bandwidth or the matrix pipe: one or two tiles per compute unit, 1 to 48
// K steps each, and a step's MFMAs (128 to 512 clocks) are shorter than a trip to L2.  So
//   * operands go straight from global memory into LDS (lds_dma.h: a wavefront instruction moves 64 x 16
//     bytes to 1 KB of consecutive LDS), NST - 1 K steps ahead, at no register cost; two stages (two to five workgroups per
//     compute unit) hide more than deeper ones;
//   * a K step is 64 wide; rows are unpadded (128 bytes) and their 16-byte pieces slot-permuted by the loading lane's
//     choice of address (piece c of row R in slot c ^ ((R >> 1) & 7)): 16-byte fragment reads of 16 consecutive rows
//     fall on 64 different banks;
//   * the stages are separate arrays and the K loop is unrolled over them: the compiler waits for every load into an LDS
//     array before any read of that array;
//   * one bare barrier per step (the fence of __syncthreads would drain the loads in flight);
//   * the residual / stored derivative / table rows a tile's epilogue needs are requested before the K loop.
// Tile 128 x 128, 64 x 128 or 64 x 64 (4 wavefronts as 2 x 2), chosen by launch_gemm_nt_mfma: larger tiles move fewer bytes per
// flop through a compute unit's L1, smaller ones reach more compute units.
// Epilogue: MFMA operands are passed swapped, so a lane holds runs of four neighbouring columns of one row; a wavefront's
// 32-row strips pass through a private LDS patch and come back as 8-column row segments: 16-byte loads and stores, each
// result rounded once - except for problems that the large-M kernels take as well (from 4,096 rows on).  Those kernels park
// a tile's results as bf16 before they add a residual or table row or multiply with the GELU derivative, and start their
// accumulators from the bias; LARGE does the same in the same order, so that which of the kernels runs does not show
// in a single bit and a slide gives the same gradients whole and in chunks.
#include "cls_lane.h"
#include "gemm_epi.h"
#include "lds_dma.h"
#include <type_traits>

namespace sl {

namespace {

constexpr int NXCD = 8;
constexpr int BK = 64;
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x8 __attribute__((ext_vector_type(8), aligned(16)));

template <int V> using IC = std::integral_constant<int, V>;

template <int N>
__device__ __forceinline__ void wait_vm() {   // until at most N vector-memory and no LDS operations of this wavefront are pending
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0070);
}

__device__ __forceinline__ void unpack8(u32x4 t, float (&v)[8]) {
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    v[2 * w] = __uint_as_float(t[w] << 16);
    v[2 * w + 1] = __uint_as_float(t[w] & 0xffff0000u);
  }
}
__device__ __forceinline__ u32x4 pack8(const float (&v)[8]) {
  bf16x8 t;
#pragma unroll
  for (int w = 0; w < 8; ++w) t[w] = (bf16)v[w];
  return __builtin_bit_cast(u32x4, t);
}

constexpr int mid_wgs(int bm, int bn, int nst) { return nst > 2 ? 1 : bm + bn == 256 ? 2 : bm + bn == 192 ? 3 : 4; }   // per compute unit

// Tile `id` of the problem.  LANE: 0, or the kernel carries a product of the CLS lane as well (1: its A is bf16, 2: float32), in its first
// workgroups; the rows of the CLS tokens are the lane's then
template <int BM, int BN, int NST, int MODE, bool LARGE, int LANE>
__device__ __forceinline__ void mid_tile(const GemmNT& g, int MT, int NTL, int id, const LaneGemm* lg, int lane_wgs, int lane_nt) {
  constexpr int WBM = BM / 64, WBN = BN / 64;        // 32 x 32 accumulators per wavefront
  constexpr int AG = BM / 32, BG = BN / 32, NLD = AG + BG;   // 8-row groups (load instructions) per wavefront and step
  constexpr int STAGE = (BM + BN) * BK;              // bf16 elements per stage
  constexpr bool HAS_BIAS = MODE == EPI_BIAS || MODE == EPI_BIAS_RESID || MODE == EPI_BIAS_GELU || MODE == EPI_TOKEN;
  constexpr bool HAS_AUX = MODE == EPI_BIAS_RESID || MODE == EPI_DGELU || MODE == EPI_ROWTAB || MODE == EPI_TOKEN;
  constexpr bool BIAS0 = LARGE && (MODE == EPI_BIAS || MODE == EPI_BIAS_RESID);   // the accumulators start from the bias
  constexpr int PS = WBN * 32 + 4;                   // patch row stride (floats)
  constexpr int SEG = WBN * 4, RPP = 64 / SEG, NP = 32 / RPP;   // 8-column segments per row, rows per pass, passes per strip
  __shared__ __attribute__((aligned(16))) bf16 st0[STAGE], st1[STAGE];
  __shared__ __attribute__((aligned(16))) bf16 st2[NST > 2 ? STAGE : 8];
  __shared__ __attribute__((aligned(16))) bf16 st3[NST > 2 ? STAGE : 8];
  static_assert(NST == 2 || NST == 4, "stages");
  static_assert(2 * 32 * PS * 4 <= STAGE * 2, "two wavefronts' epilogue patches lie inside a stage");
  // tile id -> (row tile, column tile): ids are dealt round-robin to the XCDs, and the column tiles of one row panel get
  // consecutive slots of one XCD (same L2)
  if constexpr (LANE != 0) {
    static_assert(STAGE * 2 >= 4 * 16 * 64 * 4, "a stage holds four wavefronts' partial blocks");
    if (id < lane_wgs) {
      const int mb = id / lane_nt;
      if (mb * 32LL < lg->n) lane_block4<LANE == 1>(*lg, mb, id % lane_nt, reinterpret_cast<float*>(st0), reinterpret_cast<float*>(st1));
      return;
    }
    id -= lane_wgs;
  }
  const int xcd = id % NXCD, slot = id / NXCD;
  const int mt = (slot / NTL) * NXCD + xcd;
  if (mt >= MT) return;
  const long long m0 = (long long)mt * BM;
  const int n0 = (slot % NTL) * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int nk = g.K / BK;

  // epilogue: this lane's row inside a pass and its 8-column segment
  const int prow = lane / SEG, n = n0 + wn * (WBN * 32) + (lane % SEG) * 8;
  const bool n_ok = n < g.N;
  const long long mw = m0 + wm * (WBM * 32);
  // eight one-byte codes / eight bf16 / eight floats
  typedef std::conditional_t<MODE == EPI_DGELU, u32x2, std::conditional_t<MODE == EPI_TOKEN, f32x8, u32x4>> aux_t;
  aux_t aux[HAS_AUX ? WBM : 1][HAS_AUX ? NP : 1];
  if constexpr (HAS_AUX) {
#pragma unroll
    for (int i = 0; i < WBM; ++i)
#pragma unroll
      for (int ps = 0; ps < NP; ++ps) {
        long long m = mw + i * 32 + ps * RPP + prow;
        if (m > g.M - 1) m = g.M - 1;               // never stored
        const int nn = n_ok ? n : 0;
        if constexpr (MODE == EPI_DGELU) aux[i][ps] = *reinterpret_cast<const aux_t*>((const unsigned char*)g.pre + m * g.ldpre + nn);
        else if constexpr (MODE == EPI_TOKEN) aux[i][ps] = *reinterpret_cast<const f32x8*>(g.pos + (size_t)((unsigned)m % (unsigned)g.rperiod) * g.N + nn);
        else if constexpr (MODE == EPI_ROWTAB) aux[i][ps] = *reinterpret_cast<const aux_t*>((const bf16*)g.resid + (long long)((unsigned)m % (unsigned)g.rperiod) * g.ldr + nn);
        else aux[i][ps] = *reinterpret_cast<const aux_t*>((const bf16*)g.resid + m * g.ldr + nn);
      }
  }

  // loads: instruction j of a wavefront fills rows (j * 4 + wave) * 8 .. + 7 of the tile; rows past the end lie outside of
  // the buffer (zeros, never stored)
  const int lr = lane >> 3, ls = lane & 7;
  const __amdgpu_buffer_rsrc_t ra = dma_rows((const bf16*)g.A + m0 * g.lda, (int)(g.M - m0 < BM ? g.M - m0 : BM), (int)g.lda, g.K);
  const __amdgpu_buffer_rsrc_t rb = dma_rows((const bf16*)g.B + (long long)n0 * g.ldb, g.N - n0 < BN ? g.N - n0 : BN, (int)g.ldb, g.K);
  int ao[AG], bo[BG];
#pragma unroll
  for (int j = 0; j < AG; ++j) {
    const int R = (j * 4 + wave) * 8 + lr;
    ao[j] = (R * (int)g.lda + (ls ^ ((R >> 1) & 7)) * 8) * 2;
  }
#pragma unroll
  for (int j = 0; j < BG; ++j) {
    const int R = (j * 4 + wave) * 8 + lr;
    bo[j] = (R * (int)g.ldb + (ls ^ ((R >> 1) & 7)) * 8) * 2;
  }
  auto stage = [&](auto sc) __attribute__((always_inline)) -> bf16* {
    constexpr int S = decltype(sc)::value;
    if constexpr (S == 0) return st0;
    else if constexpr (S == 1) return st1;
    else if constexpr (S == 2) return st2;
    else return st3;
  };
  auto issue = [&](auto sc, int kt) __attribute__((always_inline)) {
    bf16* s = stage(sc);
#pragma unroll
    for (int j = 0; j < AG; ++j) dma16(ra, s + (j * 4 + wave) * 8 * BK, ao[j], kt * BK * 2);
#pragma unroll
    for (int j = 0; j < BG; ++j) dma16(rb, s + BM * BK + (j * 4 + wave) * 8 * BK, bo[j], kt * BK * 2);
  };

  f32x16 acc[WBM][WBN];
#pragma unroll
  for (int j = 0; j < WBN; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4 b = {0.f, 0.f, 0.f, 0.f};
      if constexpr (BIAS0) {   // columns of accumulator elements 4q .. 4q + 3 (past the matrix: never stored)
        const int c = n0 + wn * (WBN * 32) + j * 32 + q * 8 + (lane >> 5) * 4;
        b = *reinterpret_cast<const f32x4*>(g.bias + (c < g.N ? c : 0));
      }
#pragma unroll
      for (int i = 0; i < WBM; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][j][4 * q + e] = b[e];
    }

  // fragment addresses: element offset of this lane's row in a stage, and its slot permutation (the same for every
  // 32-row block: 32 rows further leaves (R >> 1) & 7 alone)
  const int frow = lane & 31, half = lane >> 5, sw = (frow >> 1) & 7;
  const int oa = (wm * (WBM * 32) + frow) * BK, ob = (BM + wn * (WBN * 32) + frow) * BK;
  auto step = [&](auto sc, int kt) __attribute__((always_inline)) {
    constexpr int S = decltype(sc)::value;
    // this step's operands have landed: at most NST - 2 younger steps are still in flight
    const int younger = nk - 1 - kt;
    if (NST > 2 && younger >= 2) wait_vm<2 * NLD>();
    else if (NST > 2 && younger >= 1) wait_vm<NLD>();
    else wait_vm<0>();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();   // ... for every wavefront, and the stage of step kt - 1 is free
    asm volatile("" ::: "memory");
    if (kt + NST - 1 < nk) issue(IC<(S + NST - 1) % NST>{}, kt + NST - 1);
    const bf16* s = stage(sc);
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      const int c = ((ks * 2 + half) ^ sw) * 8;
      bf16x8 fa[WBM], fb[WBN];
#pragma unroll
      for (int i = 0; i < WBM; ++i) fa[i] = *reinterpret_cast<const bf16x8*>(s + oa + i * 32 * BK + c);
#pragma unroll
      for (int j = 0; j < WBN; ++j) fb[j] = *reinterpret_cast<const bf16x8*>(s + ob + j * 32 * BK + c);
#pragma unroll
      for (int i = 0; i < WBM; ++i)
#pragma unroll
        for (int j = 0; j < WBN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    }
  };
  issue(IC<0>{}, 0);
  if (NST > 2 && nk > 1) issue(IC<1>{}, 1);
  if (NST > 2 && nk > 2) issue(IC<2>{}, 2);
  int kt = 0;
  for (; kt + NST <= nk; kt += NST) {
    step(IC<0>{}, kt);
    step(IC<1>{}, kt + 1);
    if constexpr (NST > 2) { step(IC<2>{}, kt + 2); step(IC<3>{}, kt + 3); }
  }
  if (kt < nk) step(IC<0>{}, kt);
  if constexpr (NST > 2) {
    if (kt + 1 < nk) step(IC<1>{}, kt + 1);
    if (kt + 2 < nk) step(IC<2>{}, kt + 2);
  }

  // accumulator element r of lane l: row l % 32, column (r / 4) * 8 + (l / 32) * 4 + r % 4 of its block
  f32x8 bias, cls;
  if (HAS_BIAS && !BIAS0) bias = *reinterpret_cast<const f32x8*>(g.bias + (n_ok ? n : 0));
  if (MODE == EPI_TOKEN) cls = *reinterpret_cast<const f32x8*>(g.cls + (n_ok ? n : 0));
  __syncthreads();   // every wavefront is done with the stages: they become the patches, each private to its wavefront
  float* patch = reinterpret_cast<float*>(wave < 2 ? st0 : st1) + (wave & 1) * (32 * PS);
#pragma unroll
  for (int i = 0; i < WBM; ++i) {
#pragma unroll
    for (int j = 0; j < WBN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(patch + frow * PS + j * 32 + q * 8 + half * 4) =
            make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
#pragma unroll
    for (int ps = 0; ps < NP; ++ps) {
      const int row = ps * RPP + prow;
      const float4* src = reinterpret_cast<const float4*>(patch + row * PS + (lane % SEG) * 8);
      float4 a = src[0], b = src[1];
      float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
      const long long m = mw + i * 32 + row;
      if (n_ok && m < g.M && !(LANE != 0 && (unsigned)m % (unsigned)g.rperiod == 0)) {
        if constexpr (MODE == EPI_TOKEN) {
          const bool first = (unsigned)m % (unsigned)g.rperiod == 0;   // the class token's row: its product is zero
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = (v[e] + (first ? cls[e] : bias[e])) + aux[i][ps][e];
        } else if (HAS_BIAS && !BIAS0) {
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] += bias[e];
        }
        if constexpr (LARGE && HAS_AUX) unpack8(pack8(v), v);   // to bf16 and back
        if constexpr (MODE == EPI_BIAS_RESID || MODE == EPI_ROWTAB) {
          float t[8];
          unpack8(aux[i][ps], t);
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] += t[e];
        }
        if constexpr (MODE == EPI_DGELU) {
          float t0[4], t1[4];
          dg8_unpack4(aux[i][ps][0], t0);
          dg8_unpack4(aux[i][ps][1], t1);
#pragma unroll
          for (int e = 0; e < 4; ++e) { v[e] *= t0[e]; v[4 + e] *= t1[e]; }
        }
        if constexpr (MODE == EPI_BIAS_GELU) {
          float d[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) gelu_both(v[e], &v[e], &d[e]);
          if (g.out2) *reinterpret_cast<u32x2*>((unsigned char*)g.out2 + m * g.ldc2 + n) =
              u32x2{dg8_pack4(d[0], d[1], d[2], d[3]), dg8_pack4(d[4], d[5], d[6], d[7])};
        }
        *reinterpret_cast<u32x4*>((bf16*)g.out + m * g.ldc + n) = pack8(v);
      }
    }
  }
}

template <int BM, int BN, int NST, int MODE, bool LARGE>
__global__ void __launch_bounds__(256, mid_wgs(BM, BN, NST)) gemm_nt_mid_k(GemmNT g, int MT, int NTL) {
  mid_tile<BM, BN, NST, MODE, LARGE, 0>(g, MT, NTL, blockIdx.x, nullptr, 0, 1);
}
template <int BM, int BN, int NST, bool LARGE, int LANE>
__global__ void __launch_bounds__(256, mid_wgs(BM, BN, NST)) gemm_nt_mid_lane_k(GemmNT g, int MT, int NTL, LaneGemm lg, int lane_wgs, int lane_nt) {
  mid_tile<BM, BN, NST, EPI_BIAS_RESID, LARGE, LANE>(g, MT, NTL, blockIdx.x, &lg, lane_wgs, lane_nt);
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

// a product of the lane that rides along
struct Beside { const LaneGemm* lg; bool a_bf16; };

template <int BM, int BN, int NST, bool LARGE>
hipError_t go(const GemmNT& g, hipStream_t s, Beside b) {
  const int MT = (int)((g.M + BM - 1) / BM), NTL = (g.N + BN - 1) / BN;
  const long long wgs = (long long)((MT + NXCD - 1) / NXCD) * NXCD * NTL;
  if (wgs >= (1LL << 31)) return hipErrorInvalidValue;
  if (b.lg) {   // its workgroups first, and a whole number for every XCD
    const int nt = b.lg->N / 32, lw = ((int)((b.lg->n + 31) / 32) * nt + NXCD - 1) / NXCD * NXCD;
    if (b.a_bf16) hipLaunchKernelGGL((gemm_nt_mid_lane_k<BM, BN, NST, LARGE, 1>), dim3((unsigned)(wgs + lw)), dim3(256), 0, s, g, MT, NTL, *b.lg, lw, nt);
    else hipLaunchKernelGGL((gemm_nt_mid_lane_k<BM, BN, NST, LARGE, 2>), dim3((unsigned)(wgs + lw)), dim3(256), 0, s, g, MT, NTL, *b.lg, lw, nt);
    return hipGetLastError();
  }
  auto run = [&](auto mode) {
    hipLaunchKernelGGL((gemm_nt_mid_k<BM, BN, NST, decltype(mode)::value, LARGE>), dim3((unsigned)wgs), dim3(256), 0, s, g, MT, NTL);
    return hipGetLastError();
  };
  switch (g.epi) {
    case EPI_PLAIN: return run(IC<EPI_PLAIN>{});
    case EPI_BIAS: return run(IC<EPI_BIAS>{});
    case EPI_BIAS_RESID: return run(IC<EPI_BIAS_RESID>{});
    case EPI_DGELU: return run(IC<EPI_DGELU>{});
    // the table form only where the large-M kernel has it too, GELU and the float32 token rows only where it does not
    case EPI_ROWTAB: if constexpr (LARGE) return run(IC<EPI_ROWTAB>{}); else return hipErrorInvalidValue;
    case EPI_BIAS_GELU: if constexpr (!LARGE) return run(IC<EPI_BIAS_GELU>{}); else return hipErrorInvalidValue;
    case EPI_TOKEN: if constexpr (!LARGE) return run(IC<EPI_TOKEN>{}); else return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

bool gemm_nt_mfma_ok(const GemmNT& g) {
  bool ok = g.K % 64 == 0 && g.N % 16 == 0 && g.lda % 8 == 0 && g.ldb % 8 == 0 && g.lda <= DMA_LD && g.ldb <= DMA_LD && aligned16(g.A) && aligned16(g.B) &&
            g.M > 0 && g.M < (1LL << 31) && g.ldc % 8 == 0 && aligned16(g.out) && g.amap.g2 == 0 &&
            sizeof(rs_bf16path_t) == 2;
  if (g.epi == EPI_BIAS_RESID || g.epi == EPI_ROWTAB) ok = ok && g.ldr % 8 == 0 && aligned16(g.resid);
  if (g.epi == EPI_BIAS_GELU) ok = ok && g.ldc2 % 8 == 0 && ((size_t)g.out2 & 7) == 0;   // 8-byte code segments
  if (g.epi == EPI_DGELU) ok = ok && g.ldpre % 8 == 0 && ((size_t)g.pre & 7) == 0;
  if (g.epi == EPI_BIAS || g.epi == EPI_BIAS_RESID || g.epi == EPI_BIAS_GELU || g.epi == EPI_TOKEN) ok = ok && aligned16(g.bias);
  if (g.epi == EPI_TOKEN) ok = ok && aligned16(g.pos) && aligned16(g.cls) && g.rperiod > 0;
  return ok && g.epi != EPI_PATCH;
}

hipError_t launch_gemm_nt_big(const GemmNT& g, hipStream_t s);
bool gemm_nt_gelu_ok(const GemmNT& g);
hipError_t launch_gemm_nt_gelu(const GemmNT& g, hipStream_t s);

namespace {

long long tiles_of(const GemmNT& g, int bm, int bn) { return ((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn); }

constexpr int CUS = 256, XCU = CUS / NXCD;   // compute units, of the chip and of an XCD

// Whether the 256 x 192 persistent kernels are the faster ones.  Their workgroups come one per compute unit, and an XCD takes whole
// row tiles, so what counts is how full the last of the rounds is that the fullest XCD needs.  us, 128 x 128 here / 256 x 192:
//   * up to 512 tiles of 128 x 128, which is one round of two per unit, those always win: QKV of 32 ViT-S tiles 12.7 / 14.1, fc2 of 96
//     32.3 / 40.8, of 48 ViT-B tiles 53.2 / 67.2;
//   * beyond, without an operand for the epilogue or with a long contraction, by the fill: QKV 0.59 21.9 / 23.7, 0.66 22.9 / 24.3, 0.69
//     equal, 0.73 28.4 / 25.4, of three rounds and more 0.64 1.03 times, 0.97 1.25 times; fc2 of ViT-B 0.60 0.81 times, 0.66 1.04, 0.69 1.27;
//   * with an operand for the epilogue (residual, derivative, table row) and K <= 768 nothing hides the epilogue of a workgroup's last
//     tile: projection of ViT-B 0.60 of two rounds 36.3 / 50.5, 0.91 of two 51.0 / 54.0, 0.80 of three 69.0 / 76.5, 0.90 of four
//     96.3 / 95.7, 0.96 of five 133 / 121, of ViT-S 0.84 of five 76.7 / 81.0, 0.90 of six 102.4 / 97.4, 0.96 of ten 177 / 157.
bool large_fills(const GemmNT& g) {
  if (tiles_of(g, 128, 128) <= 2 * CUS) return false;
  const long long mt = (g.M + 255) / 256, nt = (g.N + 191) / 192, rounds = ((mt + NXCD - 1) / NXCD * nt + XCU - 1) / XCU;
  const long long fill = mt * nt * 100 / (rounds * CUS);   // per cent
  const bool aux = g.epi == EPI_BIAS_RESID || g.epi == EPI_DGELU || g.epi == EPI_ROWTAB;
  if (aux && g.K <= 768) return rounds >= 6 || (rounds >= 4 && fill >= 95);
  return rounds >= 3 || fill >= 67;
}

// The largest tile that gives every compute unit work, by what a unit gets: 128 x 128 from the second per unit on but for a
// nearly empty second round (two fit a unit), 64 x 128 from the fourth 64 x 64 per unit on.  us, 64 x 64 / 64 x 128 / 128 x 128,
// fc2 of 41 ViT-S tiles (762 of 64 x 64) 21.8 / 23.1 / 24.6, 42 (780) 28.8 / 23.2 / 24.9, 52 (243 of 128 x 128) 30.2 / 24.0 / 25.4, 56
// (261) 33.5 / 29.0 / 26.7, 80 (372) 42.8 / 37.1 / 30.5, 88 (408) 46.2 / 46.5 / 31.7; projection of ViT-B 444 23.5 (64 x 128) / 19.1,
// 522 25.1 / 27.8, 594 26.6 / 27.9, 744 32.0 / 29.6.  The GELU by formula keeps a workgroup's vector unit busy: 300 tiles 13.9 (64 x 128) / 15.5, 600
// 33.1 / 34.0, 744 the same.
template <bool LARGE>
hipError_t go_mid(const GemmNT& g, hipStream_t s, Beside b = {}) {
  const long long t = tiles_of(g, 128, 128);
  const bool big = g.epi == EPI_BIAS_GELU ? t >= 740 : t > CUS && (t <= 2 * CUS || t >= 5 * CUS / 2);
  if (big) return go<128, 128, 2, LARGE>(g, s, b);
  const long long t64 = tiles_of(g, 64, 64);
  if (t64 > 3 * CUS) return go<64, 128, 2, LARGE>(g, s, b);
  if (t64 <= 2 * CUS && g.K >= (t64 <= CUS ? 256 : 2048)) return go<64, 64, 4, LARGE>(g, s, b);
  return go<64, 64, 2, LARGE>(g, s, b);
}

}  // namespace

// Which kernel takes a problem: the large-M kernels where they are the faster ones, else the largest tile that gives every compute
// unit work (two workgroups of 128 x 128 fit a unit, three of 64 x 128, five of 64 x 64).
// Where there is no more than one tile a unit the chain of K steps is all that counts: four stages there (1,576 rows (150 workgroups): the
// products over K = 384, 1152 and 1536 13.0 -> 9.2 us on average; ViT-S step of 8 tiles 2174 -> 1996 us, ViT-B features of one 1117 ->
// 1043), and up to two tiles a unit if it is long (K = 3072: 17.9 us against 23.8 with two).  Elsewhere two stages and more workgroups
// measured faster.
// The GELU of the large-M kernel comes from a table whose last bits a formula does not give: that kernel has every problem it
// can take.
hipError_t launch_gemm_nt_mfma(const GemmNT& g, hipStream_t s) {
  if (gemm_nt_gelu_ok(g)) return launch_gemm_nt_gelu(g, s);
  if (!gemm_nt_big_ok(g)) return go_mid<false>(g, s);
  return large_fills(g) ? launch_gemm_nt_big(g, s) : go_mid<true>(g, s);
}

// Whether the product would run here, and not on the large-M kernels, with the lane's in its 32 x 32 form.
bool gemm_nt_lane_ok(const GemmNT& g, const LaneGemm& lg, bool a_bf16) {
  return g.epi == EPI_BIAS_RESID && g.rperiod > 0 && g.M <= LANE_BESIDE_ROWS && gemm_nt_mfma_ok(g) && !(gemm_nt_big_ok(g) && large_fills(g)) && lane_small(lg) &&
         lane_gemm_ok(lg, false, a_bf16);
}
hipError_t launch_gemm_nt_lane(const GemmNT& g, const LaneGemm& lg, bool a_bf16, hipStream_t s) {
  return gemm_nt_big_ok(g) ? go_mid<true>(g, s, {&lg, a_bf16}) : go_mid<false>(g, s, {&lg, a_bf16});
}

}  // namespace sl
