// bf16 MFMA weight-gradient GEMM for gfx950, small and medium M: C[N1,N2] = sum_m A[m,N1]^T B[m,N2] (fp32 partials).
//
// The large-M kernel (gemm_tn_big.hip) takes whole slides; this one bags of up to some 240 tiles, the CLS rows of the
// last block, narrow encoders and the aggregator.  128 x 128 of the result per workgroup (4 wavefronts as 2 x 2), M split
// into slabs.  A 32-row step moves 16 KB for 256 clocks of MFMAs, the 64 bytes a clock that a compute unit gets from its
// L2, and one trip there takes thousands of clocks: what bounds the kernel is how much a compute unit keeps in flight.
//   * operands go straight from global memory into LDS (lds_dma.h: a wavefront instruction moves 4 rows x 256
//     bytes) one step ahead at no register cost; three workgroups share a compute unit (deeper rings with fewer workgroups
//     measured 5 to 20 % slower at every size, as did 64-row steps);
//   * rows stay row-major; the MFMA operands, eight consecutive rows of one column per lane, are LDS transpose reads
//     (ds_read_b64_tr_b16: 16 lanes address 4 rows x 32 bytes).  The rows are 256 bytes apart, all on the same banks, so the
//     32-byte pieces of a row are slot-permuted by the loading lane's choice of address (piece p of row r in slot
//     p ^ 2 (r % 4)): the eight pieces that are served together fall on 64 different banks;
//   * the stages are separate arrays: the compiler waits for every load into an LDS array before any read of that array;
//   * rows past the slab's end and columns past the matrix lie outside of the buffers: zeros.
// Column sums of A (bias gradients) are taken from the operand registers by the workgroups of the first tile column: the 16
// rows a lane sees in a step first, then the even and the odd steps.
// Measured, M = 7289 (37 tiles of 197 tokens), against the kernel that transposed 8 x 8 blocks in registers on the way into
// LDS: 384 x 1536 34.9 -> 22.4 us, 1536 x 384 35.9 -> 19.5, 1152 x 384 31.9 -> 19.4, 384 x 384 14.6 -> 10.7.
#include "slide_internal.h"
#include "lds_dma.h"

namespace sl {

namespace {

constexpr long long SLOTS = 1024, CHAIN = 5280;   // workgroups of a round of the chip; rows of a slab
constexpr int BT = 128, BK = 32, STAGE = BK * 2 * BT;   // bf16 elements: [32 rows][128 columns] of A, then of B
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// problems of one launch: workgroups block0 .. of problem i, row tiles of the result innermost, then column tiles, then slabs
struct TnGroup {
  struct Prob {
    const bf16 *A, *B;
    long long lda, ldb, M;
    float *part, *cs_part;
    int N1, N2, per, block0;
  };
  int n, blocks, each;   // workgroups; those of one XCD
  Prob p[TN_GROUP_MAX];
};

__global__ void __launch_bounds__(256, 3) gemm_tn_mfma_k(TnGroup G) {
  __shared__ __attribute__((aligned(16))) bf16 st0[STAGE], st1[STAGE];
  // Workgroups are dealt round-robin to the XCDs: each XCD takes a run of consecutive ones, which are tiles of the same rows, so that
  // its L2 fetches a panel once for all the tiles of it.  The four problems of a ViT-S block, 37 tiles: 48.9 us tile by tile over the
  // XCDs, this way 43.8 (steps of 37 / 64 tiles 3276 / 4627 -> 3187 / 4455; of 4 to 8 within 0.5 % either way).
  const int wg = (int)(blockIdx.x & 7) * G.each + (int)(blockIdx.x >> 3);
  if (wg >= G.blocks) return;
  int pi = 0;
  while (pi + 1 < G.n && wg >= G.p[pi + 1].block0) ++pi;
  const TnGroup::Prob& g = G.p[pi];
  const int per = g.per, ti = (g.N1 + BT - 1) / BT, b = wg - g.block0;
  const int i0 = b % ti * BT, r = b / ti, tj = (g.N2 + BT - 1) / BT, j0 = r % tj * BT, slab = r / tj;
  const long long lo = (long long)slab * per, hi = lo + per < g.M ? lo + per : g.M;
  const int span = hi > lo ? (int)(hi - lo) : 0, nk = (span + BK - 1) / BK;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  // loads: instruction j of a wavefront fills rows (j * 4 + wave) * 4 .. + 3 of a stage; lane: row lane / 16, slot lane % 16
  const int lr = lane >> 4, lc = (((lane & 15) >> 1) ^ (2 * lr)) * 16 + (lane & 1) * 8;   // column of this lane's slot
  const int ao = i0 + lc < g.N1 ? ((wave * 4 + lr) * (int)g.lda + lc) * 2 : DMA_ABSENT;   // N1, N2 are multiples of 8
  const int bo = j0 + lc < g.N2 ? ((wave * 4 + lr) * (int)g.ldb + lc) * 2 : DMA_ABSENT;
  auto issue = [&](bf16* s, int kt) __attribute__((always_inline)) {
    const int rows = span - kt * BK < BK ? span - kt * BK : BK;
    const __amdgpu_buffer_rsrc_t ra = dma_rows(g.A + (lo + kt * BK) * g.lda + i0, rows, (int)g.lda, g.N1 - i0);
    const __amdgpu_buffer_rsrc_t rb = dma_rows(g.B + (lo + kt * BK) * g.ldb + j0, rows, (int)g.ldb, g.N2 - j0);
#pragma unroll
    for (int j = 0; j < BK / 16; ++j) {
      dma16(ra, s + (j * 4 + wave) * 4 * BT, ao, j * 32 * (int)g.lda);
      dma16(rb, s + BK * BT + (j * 4 + wave) * 4 * BT, bo, j * 32 * (int)g.ldb);
    }
  };

  // transpose reads: lane l gets column c0 + l % 32 and rows 8 (l / 32) + {0..7} of a 16-row slice
  const int gq = lane >> 4, q = lane & 15;
  auto frag_off = [&](int c0) __attribute__((always_inline)) {
    return (8 * (gq >> 1) + (q >> 2)) * BT + (((c0 >> 4) + (gq & 1)) ^ (2 * (q >> 2))) * 16 + (q & 3) * 4;
  };
  int oa[2], ob[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    oa[i] = frag_off(wm * 64 + i * 32);
    ob[i] = BK * BT + frag_off(wn * 64 + i * 32);
  }
  auto frag = [&](const bf16* p) __attribute__((always_inline)) {
    s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p);
    s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p + 4 * BT));
    s16x8 r = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    return r;
  };

  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  const bool do_cs = g.cs_part != nullptr && j0 == 0 && wn == 0;   // uniform per wavefront
  float cs0[2] = {0.f, 0.f}, cs1[2] = {0.f, 0.f};

  auto step = [&](const bf16* s, bf16* next, int kt, float (&cs)[2]) __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(0x0070);   // this wavefront's loads into LDS have landed, its LDS reads are done
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();         // ... every wavefront's
    asm volatile("" ::: "memory");
    if (kt + 1 < nk) issue(next, kt + 1);
    float c16[2] = {0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      s16x8 fa[2], fb[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        fa[i] = frag(s + oa[i] + ks * 16 * BT);
        fb[i] = frag(s + ob[i] + ks * 16 * BT);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fa[i]), __builtin_bit_cast(bf16x8, fb[j]),
                                                              acc[i][j], 0, 0, 0);
      if (do_cs) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const u32x4 t = __builtin_bit_cast(u32x4, fa[i]);
#pragma unroll
          for (int w = 0; w < 4; ++w) c16[i] += __uint_as_float(t[w] << 16) + __uint_as_float(t[w] & 0xffff0000u);
        }
      }
    }
    cs[0] += c16[0];
    cs[1] += c16[1];
  };
  if (nk > 0) issue(st0, 0);
  int kt = 0;
  for (; kt + 2 <= nk; kt += 2) {
    step(st0, st1, kt, cs0);
    step(st1, st0, kt + 1, cs1);
  }
  if (kt < nk) step(st0, st1, kt, cs0);

  if (do_cs) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      float cs = cs0[i] + cs1[i];
      cs += __shfl_xor(cs, 32, 64);
      const int c = i0 + wm * 64 + i * 32 + (lane & 31);
      if (lane < 32 && c < g.N1) g.cs_part[(size_t)slab * g.N1 + c] = cs;
    }
  }
  float* P = g.part + (size_t)slab * g.N1 * g.N2;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      int c = j0 + wn * 64 + j * 32 + (lane & 31);
      bool c_ok = c < g.N2;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        int row = i0 + wm * 64 + i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
        if (c_ok && row < g.N1) P[(size_t)row * g.N2 + c] = acc[i][j][r];
      }
    }
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace

bool gemm_tn_mfma_ok(const GemmTN& g) {
  return g.N1 % 8 == 0 && g.N2 % 8 == 0 && g.lda % 8 == 0 && g.ldb % 8 == 0 && g.lda <= DMA_LD && g.ldb <= DMA_LD && aligned16(g.A) && aligned16(g.B) &&
         g.amap.g2 == 0 && g.bmap.g2 == 0 && g.M < (1LL << 31);
}

// Rows of a slab, for problems that run as one launch: about two workgroups per compute unit over all of them, no slab of less
// than 128 rows (64 where there are only a few tiles), since every slab's result is written and read again.  M = 7289, 384 x
// 1536 alone (36 tiles), us: 4 slabs 33, 8 22.8, 11 22.4, 15 22.8, 29 28.3; 384 x 384: 15 slabs 12.6, 29 10.7, 57 11.9; M =
// 1000, 1536 x 384: 8 slabs 8.7, 16 10.4.  Step of 37 ViT-S tiles, the four problems of a block together, by workgroups: 384 3.24
// ms, 512 3.19, 768 3.21.
// From 1,400 rows in each on as many slabs as fill whole rounds of the four workgroups that a unit holds, of 5,280 rows at most (a
// slab is one chain of float32 additions).  ViT-S steps, ms, by two a unit / this way: 80 tiles 5.07 / 4.99, 135 7.85 / 7.67, 200 10.79 /
// 10.49; ten slabs of 108 tiles (1,080 workgroups) 13.9 at 256 tiles, where eighteen take 12.98.
void gemm_tn_mfma_slabs(GemmTN* g, int n, int max_slabs) {
  long long work = 0, tiles = 0;   // rows x tiles
  for (int i = 0; i < n; ++i) {
    const long long t = (long long)((g[i].N1 + BT - 1) / BT) * ((g[i].N2 + BT - 1) / BT);
    work += t * g[i].M;
    tiles += t;
  }
  long long per = (work + 511) / 512, least = tiles <= 8 ? 64 : 128;
  if (per < least) per = least;
  const long long rows = work / tiles;
  for (long long r = 1; r <= 8; ++r) {   // rounds
    const long long slabs = SLOTS * r / tiles;
    if (slabs < 1) continue;
    const long long p = (rows + slabs - 1) / slabs;
    if (r == 1 && p < 1400) break;
    per = p;
    if (p <= CHAIN) break;
  }
  for (int i = 0; i < n; ++i) {
    long long s = (g[i].M + per - 1) / per;
    if (s > max_slabs) s = max_slabs;
    g[i].slabs = s < 1 ? 1 : (int)s;
  }
}

hipError_t launch_gemm_tn_mfma(const GemmTN* g, int n, hipStream_t s) {
  if (n < 1 || n > TN_GROUP_MAX) return hipErrorInvalidValue;
  TnGroup G;
  G.n = n;
  long long blocks = 0;
  for (int i = 0; i < n; ++i) {
    TnGroup::Prob& p = G.p[i];
    p.A = (const bf16*)g[i].A; p.lda = g[i].lda; p.B = (const bf16*)g[i].B; p.ldb = g[i].ldb; p.M = g[i].M;
    p.N1 = g[i].N1; p.N2 = g[i].N2; p.part = g[i].part; p.cs_part = g[i].cs_part;
    p.per = (int)(((g[i].M + g[i].slabs - 1) / g[i].slabs + BK - 1) / BK * BK);
    p.block0 = (int)blocks;
    blocks += (long long)((p.N1 + BT - 1) / BT) * ((p.N2 + BT - 1) / BT) * g[i].slabs;
  }
  if (blocks >= (1LL << 31) - 8) return hipErrorInvalidValue;
  G.blocks = (int)blocks;
  G.each = (int)((blocks + 7) / 8);
  hipLaunchKernelGGL(gemm_tn_mfma_k, dim3((unsigned)G.each * 8), dim3(256), 0, s, G);
  return hipGetLastError();
}

}  // namespace sl
