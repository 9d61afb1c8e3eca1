// The MLP half of a transformer block in one kernel (bf16, D = 384): out = x + gelu(LN(x) W1^T + b1) W2^T + b2, and its
// backward h = (A W1^T) * gelu', out = h W2^T (W1, W2 then the transposed copies of fc2 and fc1).
//
// As two GEMMs the hidden layer goes through memory: 3072 bytes a row out and in again beside 768 in and 768 out, and the
// K = 384 product spends more time on its epilogue than on its MFMAs.  Here a wavefront keeps everything that belongs to its
// 32 rows in registers and only the weights move:
//   * 4 wavefronts per workgroup, one per SIMD with 512 registers: the rows of A as fragments (96), the output's
//     accumulators (12 blocks of 32 x 32 = 192), the hidden layer of 64 columns (32, and 32 while it is activated).
//   * Both products run transposed, H^T = W1 A^T and out^T += W2 H^T: a lane then holds four consecutive hidden columns of
//     one row, and two v_permlane32_swap turn eight packed values into the fragment the second product wants.  The hidden
//     layer never leaves the wavefront, so the wavefronts meet only at the weights.
//   * The weights stream through four stages of 24 KB in LDS (buffer_load ... lds, 16 bytes a lane; the buffer form, because
//     behind a global_load ... lds the compiler waits for all LDS reads at every one), requested three stages ahead; one bare
//     barrier per 24 MFMAs, six MFMAs before the stage's end, so that the first fragments of the next stage arrive under them.
//     128 bytes of rows are slot-permuted as in gemm_nt_mfma.hip.
//   * The activation of step s runs between the MFMAs of the second product of step s - 1 and the first of step s + 1, one
//     element per three MFMAs, in explicit order (a fence per MFMA).
//   * The forward's LayerNorm is taken on the rows in their registers (a row is two lanes'), at a tile's end for the next one, while
//     the tile's results are on their way out.  As a launch of its own it read and wrote every row once more: features of 3001 ViT-S
//     tiles 38.8 -> 37.9 ms.
// K order, initial bias, table, the LayerNorm's order of additions and every rounding are those of the large-M GEMM and the LayerNorm
// kernels, so the results are theirs bit for bit (whole slides and chunks take different kernels).
//
// What bounds it: the matrix pipe is busy half of the clocks (49 % forward, 46 % backward at 2.0 GHz); each MFMA takes one
// fragment from LDS (fragments for every second one only: -14 % of the loop), the activation's instructions share the issue
// with it (without: -15 %), and the weights are 96 KB per step and compute unit of L1 fill (without: -14 %).  Rows and results of a
// tile, 288 KB, move at its end in a burst of all compute units: 0.25 of 1.43 ms at 591,197 rows.
// 591,197 rows, F = 1536, two launches / here: forward without a backward to come 1.77 / 1.43 ms (0.98 PFLOP/s), backward 1.77 / 1.55 ms.
// A forward that also stores the hidden layer and the derivative's codes was tried in this form: 2.00 / 1.90 ms with many
// rounds of workgroups and slower with two or three (h stores of 24 KB per step and unit share the L1's queue with the weights'
// loads), so that case stays two launches.  Tried besides: stores spread over the step (slower: each is waited for with
// the weight loads behind it, and vmcnt is in order), weight loads split between wavefronts by stage (no change), fragments
// read two to four at a time (no change).
#include "slide_internal.h"

#include <type_traits>

namespace sl {

namespace {

constexpr int D = 384;                 // width of the rows
constexpr int NW = 4, NTH = 64 * NW;   // wavefronts per workgroup: one per SIMD, 512 registers each
constexpr int RW = 32, RB = NW * RW;   // rows per wavefront and workgroup
constexpr int FS = 64;                 // hidden columns per step
constexpr int UNIT = 192 * 64;         // bf16 elements per stage of the weight ring (24 KB)
constexpr int NM = 24;                 // MFMAs per wavefront and stage
constexpr int FR = 8;                  // fragment registers
constexpr int AHEAD = 6;               // fragments read ahead
constexpr int BAR = NM - AHEAD;        // the MFMA before which a stage's barrier sits
constexpr int ND = 6;                  // loads of a wavefront per stage
constexpr int PB = 400;                // patch row stride (bytes): 192 bf16 and a pad
constexpr int TAB_N = 448;             // table over [-7, 7) in steps of 1/32, as in gemm_nt_gelu.hip
constexpr int F_MAX = 1536;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 h16x2 __attribute__((ext_vector_type(2)));
typedef void __attribute__((address_space(3)))* lptr_t;

template <int V> using IC = std::integral_constant<int, V>;

template <int N>
__device__ __forceinline__ void wait_vm() {   // until at most N vector-memory operations of this wavefront are pending
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0f70);
}

__device__ __forceinline__ unsigned pack2(float a, float b) {
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  b2 t = {(bf16)a, (bf16)b};
  return __builtin_bit_cast(unsigned, t);
}
// the upper half of a against the lower half of b; rows of 16 lanes: the odd ones of a against the even ones of b
__device__ __forceinline__ void swap32(unsigned& a, unsigned& b) {
  auto t = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = t[0];
  b = t[1];
}
__device__ __forceinline__ void swap16(u32x4& a, u32x4& b) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    auto t = __builtin_amdgcn_permlane16_swap(a[i], b[i], false, false);
    a[i] = t[0];
    b[i] = t[1];
  }
}

enum { A_UNIT = 0, B_UNIT = 1 };
// of 48 slots (MFMAs): the one in which the activation of element e of 16 begins; its table entry is used ACT_LAT later
__device__ __host__ constexpr int act_slot(int e) { return e * 11 / 4; }
constexpr int ACT_LAT = 6;

// GRAD: the backward form
template <bool GRAD>
__global__ void __launch_bounds__(NTH, 1) mlp_k(MlpArgs g, int tiles) {
  __shared__ __attribute__((aligned(16))) bf16 st0[UNIT], st1[UNIT], st2[UNIT], st3[UNIT];
  __shared__ __attribute__((aligned(16))) unsigned char patches[NW * RW * PB];
  __shared__ __attribute__((aligned(16))) float lb1[GRAD ? 4 : F_MAX], lb2[GRAD ? 4 : D];
  __shared__ __attribute__((aligned(16))) float lgam[GRAD ? 4 : D], lbet[GRAD ? 4 : D];
  __shared__ h16x2 tab[GRAD ? 1 : TAB_N];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, frow = lane & 31, sw = (frow >> 1) & 7;
  const int ns = g.F / FS;   // steps, three at least
  int tile = blockIdx.x;
  if (tile >= tiles) return;
  if constexpr (!GRAD) {
    for (int k = tid; k < TAB_N; k += NTH) {
      float x0 = -7.0f + (float)k * (1.0f / 32.0f), x1 = x0 + (1.0f / 32.0f);
      float c0 = 0.5f * (1.0f + erff(x0 * 0.70710678118654752f)), c1 = 0.5f * (1.0f + erff(x1 * 0.70710678118654752f));
      tab[k] = h16x2{(_Float16)c0, (_Float16)(c1 - c0)};
    }
    for (int k = tid; k < g.F; k += NTH) lb1[k] = g.b1[k];
    for (int k = tid; k < D; k += NTH) { lb2[k] = g.b2[k]; lgam[k] = g.gam[k]; lbet[k] = g.bet[k]; }
  }

  auto stage = [&](auto sc) __attribute__((always_inline)) -> bf16* {
    constexpr int S = decltype(sc)::value;
    if constexpr (S == 0) return st0;
    else if constexpr (S == 1) return st1;
    else if constexpr (S == 2) return st2;
    else return st3;
  };
  // ---- weight ring
  const __amdgpu_buffer_rsrc_t r1 = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.W1), 0, 2 * D * g.F, 0x00027000);
  const __amdgpu_buffer_rsrc_t r2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.W2), 0, 2 * D * g.F, 0x00027000);
  const int piece = (lane & 7) ^ ((wave & 1) * 4 + (lane >> 4));
  const int la = (lane >> 3) * (2 * D) + piece * 16 + wave * 8 * 2 * D;
  const int lb = (lane >> 3) * (2 * g.F) + piece * 16 + wave * 8 * 2 * g.F;
  auto dma = [&](auto sc, auto kind, auto hc, int s, int j) __attribute__((always_inline)) {
    bf16* st = stage(sc) + (j * 4 + wave) * 512;
    if constexpr (decltype(kind)::value == A_UNIT) {
      const int o = s * (FS * 2 * D) + decltype(hc)::value * 384 + (j >> 1) * 128 + (j & 1) * (4 * 8 * 2 * D);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r1, (lptr_t)st, 16, la, o, 0, 0);
    } else {
      const int o = s * (FS * 2) + (decltype(hc)::value * 192 + j * 32) * 2 * g.F;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r2, (lptr_t)st, 16, lb, o, 0, 0);
    }
  };
  // ---- rows of a tile: loads past the end give zeros, stores past it are dropped
  auto rows_of = [&](const void* p, int t, int row_bytes) __attribute__((always_inline)) {
    const long long m0 = (long long)t * RB;
    const int rows = g.M - m0 > RB ? RB : g.M - m0 > 0 ? (int)(g.M - m0) : 0;
    return __builtin_amdgcn_make_buffer_rsrc((char*)const_cast<void*>(p) + m0 * row_bytes, 0, rows * row_bytes, 0x00027000);
  };
  const int row0 = wave * RW;
  const int uoff = (row0 + frow) * (2 * D) + half * 16;
  // 16-byte piece p * 64 + lane of a wavefront's 32 rows x 192 columns, 24 a row; three passes are eight rows
  int qoff[3], loff[3];
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    const int i = p * 64 + lane, r = i / 24, c = i % 24;
    qoff[p] = (row0 + r) * (2 * D) + c * 16;
    loff[p] = r * PB + c * 16;
  }
  // stores of the hidden layer: after swap16 lane l holds row l % 16 (or 16 more)
  const int hoff = (row0 + (lane & 15)) * 2 * g.F + (((lane >> 4) & 1) * 32 + (lane >> 5) * 16);
  const int coff = (row0 + (lane & 15)) * g.F + (lane >> 4) * 16;

  // stores of the hidden layer in the first B stage of a step, loads of derivative codes in its first A stage
  constexpr int P0 = GRAD ? 4 : 0, NLD = GRAD ? 2 : 0;
  // ---- registers
  f32x16 Y[12], H[2];
  bf16x8 U[24], fr[FR];
  u32x4 pk[4], cd[2], ht[2];
  unsigned cc[8];
  float x[32], ff[4];
  h16x2 te[4];
  __amdgpu_buffer_rsrc_t rh, rc;

  int oc[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) oc[k] = frow * 64 + ((k * 2 + half) ^ sw) * 8;
  auto rd = [&](auto sc, auto kind, int n) __attribute__((always_inline)) {
    const bf16* st = stage(sc);
    if constexpr (decltype(kind)::value == A_UNIT) {
      const int ks = n >> 1, fb = n & 1;
      fr[n % FR] = *reinterpret_cast<const bf16x8*>(st + (ks >> 2) * 4096 + fb * 2048 + oc[ks & 3]);
    } else {
      const int ks = n / 6, db = n % 6;
      fr[n % FR] = *reinterpret_cast<const bf16x8*>(st + db * 2048 + oc[ks]);
    }
  };
  auto take = [&](int e) __attribute__((always_inline)) {   // an accumulator into a register of its own, here and not later
    x[e] = H[e >> 4][e & 15];
    asm volatile("" : "+v"(x[e]));
  };
  auto act_start = [&](int e) __attribute__((always_inline)) {
    if constexpr (!GRAD) {
      float t = __builtin_amdgcn_fmed3f(x[e] * 32.0f + 224.0f, 0.0f, (float)TAB_N - 0.001f);
      te[e & 3] = tab[(int)t];
      ff[e & 3] = __builtin_amdgcn_fractf(t);
    }
  };
  auto act_end = [&](int e) __attribute__((always_inline)) {
    if constexpr (GRAD) {
      const unsigned b = (cc[e >> 2] >> (8 * (e & 3))) & 0xffu;
      x[e] = (float)(bf16)x[e] * ((float)b * (1.0f / DG8_SCALE) - DG8_OFF);
    } else {
      x[e] = x[e] * ((float)te[e & 3][0] + ff[e & 3] * (float)te[e & 3][1]);
    }
  };
  auto pack_ks = [&](int ks) __attribute__((always_inline)) {
    const float* v = x + ks * 8;
    unsigned p0 = pack2(v[0], v[1]), p1 = pack2(v[2], v[3]), q0 = pack2(v[4], v[5]), q1 = pack2(v[6], v[7]);
    swap32(p0, q0);
    swap32(p1, q1);
    pk[ks] = u32x4{p0, p1, q0, q1};
  };
  auto h_init = [&](int fb, int q, int s) __attribute__((always_inline)) {
    if constexpr (GRAD) {
#pragma unroll
      for (int e = 0; e < 4; ++e) H[fb][4 * q + e] = 0.f;
    } else {
      float4 b = *reinterpret_cast<const float4*>(lb1 + s * FS + fb * 32 + q * 8 + half * 4);
      H[fb][4 * q] = b.x; H[fb][4 * q + 1] = b.y; H[fb][4 * q + 2] = b.z; H[fb][4 * q + 3] = b.w;
    }
  };
  // the stored hidden layer, two K slices at a time: 64 contiguous bytes of 16 rows per instruction
  auto put_h = [&](int s, int i) __attribute__((always_inline)) {
    if (!(i & 1)) {
      ht[0] = pk[i];
      ht[1] = pk[i + 1];
      swap16(ht[0], ht[1]);
    }
    __builtin_amdgcn_raw_buffer_store_b128(ht[i & 1], rh, hoff, s * (FS * 2) + (i >> 1) * 64 + (i & 1) * 32 * g.F, 0);
  };
  auto load_c = [&](int s, int i) __attribute__((always_inline)) {
    cd[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rc, coff, s * FS + i * 16 * g.F, 0));
  };
  auto open_c = [&]() __attribute__((always_inline)) {
    swap16(cd[0], cd[1]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      unsigned a = cd[j >> 1][(j & 1) * 2], b = cd[j >> 1][(j & 1) * 2 + 1];
      swap32(a, b);
      cc[j] = a;
      cc[j + 4] = b;
    }
  };

  // One stage: 24 MFMAs out of ring stage sc, half hc of step s0's first (A) or second (B) product; nkind: the stage behind
  // it.  Behind the barrier the stage three further on (kind k3, half h3, step s3) is requested.  younger: vector-memory
  // operations, beside that stage's, that are certainly issued after the loads of the next one (counting too few waits too long, never too
  // short).  act: the activation of 16 elements rides along (B: x[0..15], A: x[16..31]); sn: the step the hidden accumulators start next
  auto unit = [&](auto sc, auto kind, auto hc, auto nkind, auto act, auto younger, auto k3, auto h3, int s3, int sn, int s0) __attribute__((always_inline)) {
    constexpr int S = decltype(sc)::value, K = decltype(kind)::value, HC = decltype(hc)::value;
    constexpr bool ACT = decltype(act)::value != 0;
    constexpr int YOUNGER = ND + decltype(younger)::value;   // vector-memory operations younger than the next stage's loads
#pragma unroll
    for (int n = 0; n < NM; ++n) {
      if (n == BAR) {
        wait_vm<YOUNGER>();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      }
      if constexpr (K == A_UNIT) {
        H[n & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[n % FR], U[HC * 12 + (n >> 1)], H[n & 1], 0, 0, 0);
      } else {
        const int d = HC * 6 + n % 6;
        Y[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[n % FR], __builtin_bit_cast(bf16x8, pk[n / 6]), Y[d], 0, 0, 0);
      }
      if (n < BAR) rd(IC<S>{}, kind, n + AHEAD);
      else rd(IC<(S + 1) % 4>{}, nkind, n - BAR);
      if (n >= BAR) dma(IC<(S + 3) % 4>{}, k3, h3, s3, n - BAR);
      const int m = HC * NM + n;   // slot of 48
      if constexpr (K == B_UNIT && GRAD) {
        if (m == 0) put_h(s0, 0);
        if (m == 0) put_h(s0, 1);
        if (m == 2) put_h(s0, 2);
        if (m == 2) put_h(s0, 3);
      }
      if constexpr (GRAD && ACT && K == A_UNIT) {
        if (m < 2) load_c(s0, m);
      }
      if constexpr (GRAD && ACT && K == B_UNIT) {
        if (m == 5) open_c();
      }
      if constexpr (ACT) {
        if (K == B_UNIT && m < 32) take((m >> 1) + (m & 1) * 16);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          if (act_slot(e) == m) act_start((K == A_UNIT ? 16 : 0) + e);
          if (act_slot(e) + ACT_LAT == m) act_end((K == A_UNIT ? 16 : 0) + e);
        }
        if constexpr (K == A_UNIT) {
          if (m == 4) pack_ks(0);
          if (m == 8) pack_ks(1);
          if (m == 26) pack_ks(2);
          if (m == 47) pack_ks(3);
        } else {
          if (m >= 36 && m < 44) h_init((m - 36) >> 2, (m - 36) & 3, sn);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  constexpr IC<0> c0{};
  constexpr IC<1> c1{};
  constexpr IC<2> c2{};
  constexpr IC<3> c3{};
  constexpr IC<A_UNIT> A{};
  constexpr IC<B_UNIT> B{};
  constexpr IC<1> yes{};
  constexpr IC<0> no{};

  auto load_u = [&](int t) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t ru = rows_of(g.A, t, 2 * D);
#pragma unroll
    for (int k = 0; k < 24; ++k) U[k] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(ru, uoff, k * 32, 0));
  };

  // LayerNorm of the rows in U, in the order of ln_fwd_row16_k: there 16 lanes share a row, lane l with its pieces l, l + 16, l + 32 of
  // eight columns; here lane half h has pieces 2 k + h, so that lane's sum is the one over k = l / 2, + 8, + 16, and the exchanges over
  // eight, four and two lanes are sums of registers
  auto norm_u = [&]() __attribute__((always_inline)) {
    auto un = [&](int k, float (&v)[8]) __attribute__((always_inline)) {
      const u32x4 t = __builtin_bit_cast(u32x4, U[k]);
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        v[2 * w] = __uint_as_float(t[w] << 16);
        v[2 * w + 1] = __uint_as_float(t[w] & 0xffff0000u);
      }
    };
    auto total = [&](float (&s)[8]) __attribute__((always_inline)) {
#pragma unroll
      for (int o = 4; o > 0; o >>= 1)
#pragma unroll
        for (int j = 0; j < o; ++j) s[j] += s[j + o];
      return s[0] + __shfl_xor(s[0], 32, 64);
    };
    // the rows are unpacked anew by every pass over them: kept unpacked they would take 192 registers
    auto again = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < 24; ++k) asm volatile("" : "+v"(U[k]));
    };
    float s[8], v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      s[j] = 0.f;
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        un(j + 8 * i, v);
#pragma unroll
        for (int e = 0; e < 8; ++e) s[j] += v[e];
      }
    }
    const float sum = total(s);
    again();
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      s[j] = 0.f;
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        un(j + 8 * i, v);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = ln_centre(v[e], sum, D);
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (i > 0 || e > 1) s[j] = fmaf(v[e], v[e], s[j]);
          else if (e == 1) s[j] = ln_squares(v[0], v[1]);
      }
    }
    const float rstd = ln_rstd(total(s), D, g.eps);
    again();
#pragma unroll
    for (int k = 0; k < 24; ++k) {
      un(k, v);
      float gb[16];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        *reinterpret_cast<f32x4*>(gb + 4 * q) = *reinterpret_cast<const f32x4*>(lgam + k * 16 + half * 8 + 4 * q);
        *reinterpret_cast<f32x4*>(gb + 8 + 4 * q) = *reinterpret_cast<const f32x4*>(lbet + k * 16 + half * 8 + 4 * q);
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) U[k][e] = (bf16)fmaf(ln_centre(v[e], sum, D) * rstd, gb[e], gb[8 + e]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  load_u(tile);
#pragma unroll
  for (int j = 0; j < 6; ++j) dma(c0, A, c0, 0, j);
#pragma unroll
  for (int j = 0; j < 6; ++j) dma(c1, A, c1, 0, j);
#pragma unroll
  for (int j = 0; j < 6; ++j) dma(c2, A, c0, 1, j);
  wait_vm<0>();   // the first stages count no younger operations
  __syncthreads();
  if constexpr (!GRAD) norm_u();
#pragma unroll
  for (int n = 0; n < AHEAD; ++n) rd(c0, A, n);

  unsigned char* const patch = patches + wave * RW * PB;
  constexpr int EDGE = GRAD ? 24 : 36;   // loads of the next tile's rows and of half of the residual's
  for (;;) {
#pragma unroll
    for (int d = 0; d < 12; ++d)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float4 b = make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (!GRAD) b = *reinterpret_cast<const float4*>(lb2 + d * 32 + q * 8 + half * 4);
        Y[d][4 * q] = b.x; Y[d][4 * q + 1] = b.y; Y[d][4 * q + 2] = b.z; Y[d][4 * q + 3] = b.w;
      }
#pragma unroll
    for (int q = 0; q < 4; ++q) { h_init(0, q, 0); h_init(1, q, 0); }
    if constexpr (GRAD) {
      rh = rows_of(g.h, tile, 2 * g.F);
      rc = rows_of(g.code, tile, g.F);
      load_c(0, 0);
      load_c(0, 1);
    }
    unit(c0, A, c0, A, no, IC<24>{}, A, c1, 1, 0, 0);
    unit(c1, A, c1, A, no, IC<24>{}, B, c0, 0, 0, 0);
    if constexpr (GRAD) open_c();
#pragma unroll
    for (int e = 0; e < 32; ++e) take(e);
#pragma unroll
    for (int e = 0; e < 16; ++e) { act_start(e); act_end(e); }
#pragma unroll
    for (int q = 0; q < 4; ++q) { h_init(0, q, 1); h_init(1, q, 1); }
    for (int s = 1; s < ns - 1; ++s) {
      unit(c2, A, c0, A, yes, IC<NLD>{}, B, c1, s - 1, 0, s);
      unit(c3, A, c1, B, yes, IC<NLD>{}, A, c0, s + 1, 0, s);
      unit(c0, B, c0, B, yes, IC<P0>{}, A, c1, s + 1, s + 1, s - 1);
      unit(c1, B, c1, A, yes, IC<P0>{}, B, c0, s, s + 1, s - 1);
    }
    unit(c2, A, c0, A, yes, IC<NLD>{}, B, c1, ns - 2, 0, ns - 1);
    unit(c3, A, c1, B, yes, IC<NLD>{}, B, c0, ns - 1, 0, ns - 1);
    const int next = tile + gridDim.x;
    unit(c0, B, c0, B, yes, IC<P0>{}, B, c1, ns - 1, 0, ns - 2);
    unit(c1, B, c1, B, yes, IC<P0>{}, A, c0, 0, 0, ns - 2);
#pragma unroll
    for (int e = 16; e < 32; ++e) { act_start(e); act_end(e); }
#pragma unroll
    for (int k = 0; k < 4; ++k) pack_ks(k);
    const __amdgpu_buffer_rsrc_t ro = rows_of(g.out, tile, 2 * D);
    u32x4 rs[2][12];
    auto load_r = [&](int h) __attribute__((always_inline)) {
      const __amdgpu_buffer_rsrc_t rr = rows_of(g.A, tile, 2 * D);
#pragma unroll
      for (int p = 0; p < 12; ++p) rs[h][p] = __builtin_amdgcn_raw_buffer_load_b128(rr, qoff[p % 3], (p / 3) * 8 * 2 * D + h * 384, 0);
    };
    if constexpr (!GRAD) load_r(0);
    load_u(next);    // past the last tile: nothing is read
    __builtin_amdgcn_sched_barrier(0);
    unit(c2, B, c0, B, no, IC<EDGE + P0>{}, A, c1, 0, 0, ns - 1);
    unit(c3, B, c1, A, no, IC<EDGE + P0>{}, A, c0, 1, 0, ns - 1);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int d = 0; d < 6; ++d)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<u32x2*>(patch + frow * PB + d * 64 + q * 16 + half * 8) =
              u32x2{pack2(Y[h * 6 + d][4 * q], Y[h * 6 + d][4 * q + 1]), pack2(Y[h * 6 + d][4 * q + 2], Y[h * 6 + d][4 * q + 3])};
      if (!GRAD && h == 0) load_r(1);
#pragma unroll
      for (int p = 0; p < 12; ++p) {
        u32x4 o = *reinterpret_cast<const u32x4*>(patch + loff[p % 3] + (p / 3) * 8 * PB);
        if constexpr (!GRAD) {
#pragma unroll
          for (int w = 0; w < 4; ++w)
            o[w] = pack2(__uint_as_float(o[w] << 16) + __uint_as_float(rs[h][p][w] << 16),
                         __uint_as_float(o[w] & 0xffff0000u) + __uint_as_float(rs[h][p][w] & 0xffff0000u));
        }
        __builtin_amdgcn_raw_buffer_store_b128(o, ro, qoff[p % 3], (p / 3) * 8 * 2 * D + h * 384, 0);
      }
    }
    if (next >= tiles) break;
    tile = next;
    if constexpr (!GRAD) norm_u();
  }
  wait_vm<0>();   // the ring's last loads land before the workgroup's LDS is given back
}

}  // namespace

namespace {

int compute_units() {
  static const int cus = [] {
    int dev = 0;
    hipDeviceProp_t prop;
    return hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess ? prop.multiProcessorCount : 256;
  }();
  return cus;
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace

bool mlp_ok(const MlpArgs& g, int width, bool grad) {
  if (!(width == D && g.F % FS == 0 && g.F >= 3 * FS && g.F <= F_MAX && g.M > 0 && g.M < (1LL << 31))) return false;
  if (!(aligned16(g.A) && aligned16(g.W1) && aligned16(g.W2) && aligned16(g.out) && aligned16(g.h) && aligned16(g.code))) return false;
  if (!grad && !(aligned16(g.b1) && aligned16(g.b2) && aligned16(g.gam) && aligned16(g.bet))) return false;
  // A workgroup takes 128 rows and comes once per compute unit, so what counts is how full the last round of them is.  Two launches /
  // here, by rounds, us forward: 0.50 60 / 72, 0.59 85 / 71, 0.84 103 / 80, 1.00 108 / 89, 1.01 130 / 140, 1.09 136 / 143, 1.15
  // 150 / 145, 1.20 152 / 145, 1.45 169 / 149, 2.00 205 / 167, 2.01 245 / 219, 3.01 332 / 290, 6.0 600 / 522; backward: 0.59 82 / 80,
  // 0.63 81 / 82, 0.68 94 / 85, 1.00 116 / 96, 1.01 143 / 157, 1.15 153 / 153, 1.27 164 / 156, 1.45 172 / 162, 2.01 244 / 235,
  // 3.01 330 / 312, 6.0 616 / 556.  The weight gradient behind the backward form takes 1 to 2 us longer than behind two launches, hence
  // its higher line: steps of 1.2 and 1.27 rounds measured the same either way, of 1.02 and less slower here.
  const long long tiles = (g.M + RB - 1) / RB, cus = compute_units(), rounds = (tiles + cus - 1) / cus;
  return tiles * 100 >= (grad ? 65 : 58) * rounds * cus;
}

hipError_t launch_mlp(const MlpArgs& g, bool grad, hipStream_t s) {
  const int tiles = (int)((g.M + RB - 1) / RB), cus = compute_units();
  const dim3 grid(tiles < cus ? tiles : cus);
  if (grad) hipLaunchKernelGGL(mlp_k<true>, grid, dim3(NTH), 0, s, g, tiles);
  else hipLaunchKernelGGL(mlp_k<false>, grid, dim3(NTH), 0, s, g, tiles);
  return hipGetLastError();
}

}  // namespace sl
