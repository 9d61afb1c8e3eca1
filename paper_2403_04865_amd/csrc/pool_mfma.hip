// Gated-attention MIL pooling, forward stage 1 on the matrix cores (gfx950, bf16 path).
//
// a_n = w . (tanh(V h_n + b_V) * sigmoid(U h_n + b_U)) needs 4 * M_h * D flop per feature row of D * 4 bytes:
// 128 flop/byte at M_h = 128, far more than the vector ALUs deliver at HBM speed, so the two projections are one
// bf16 MFMA GEMM [rows] x [V;U]^T with fp32 accumulation.  Everything else stays fp32 / fp64 on the
// unrounded features: the softmax over tiles is a two-level online reduction (every workgroup keeps a running
// max, sum and weighted feature sum over its row blocks; one workgroup combines them afterwards).
// Two kernels:
//   * pool_gate_part_reg_k (D = 384, M_h = 128; M_h = 256 as two halves of the gate units, side by side or one after the other): the main
//     one.  One persistent workgroup (4 wavefronts) per compute unit; the bf16 copy of
//     [V;U] is 192 kB, which is what the accumulation half of a compute unit's register file holds, so every
//     wavefront keeps the fragments of its 32 gate units in registers for the whole kernel and the only traffic is
//     the feature rows, each read from HBM exactly once into fp32 registers (a bf16 image in LDS feeds the MFMAs;
//     the weighted feature sum is taken from the unrounded registers).  The gate arithmetic of block i - 1 is
//     issued between the MFMAs of block i.
//   * pool_gate_part_stream_k (D = 768): the weights are more than the registers hold and stream from L2, straight into fragments.
//   Operands are passed swapped (weights first): a lane then owns one feature row and 16 gate units per
//   accumulator, so the sum over gate units is in-lane plus one exchange between the lane halves.
#include "slide_internal.h"
#include "split_f32.h"

namespace sl {

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

template <int V>
struct IC { static constexpr int value = V; };
template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(IC<I>{});
    static_for<I + 1, N>(f);
  }
}

// [V;U] of 128 gate units x D as the kernels take them: every wavefront load of a fragment is 1 KB in a row
// (row-major, the lanes of a load touch 32 rows, which fills a compute unit's L1 at a third of the rate: 192 KB in 5 us
// against 2).  Half h of the gate units (units 128 h .. + 127) at out + h * 2 * FRAG: FRAG elements of [V;U], for wavefront w,
// slice ks, matrix m the 64 lanes' eight values (unit 32 w + l % 32, column 16 ks + 8 (l / 32) ..); then, if transposed, FRAG
// elements of its transpose (column 32 b + l % 32, unit 16 ks + 8 (l / 32) .. of V's 128 and U's 128).  The second half starts at the same
// place without transposes, so `out` has room for both copies in every call.
constexpr int FRAG_D = 384, FRAG_MH = 128;
constexpr int frag(int D) { return 2 * FRAG_MH * D; }
template <int D>
__global__ void __launch_bounds__(256) pool_cast_frag_k(const float* __restrict__ V, const float* __restrict__ U, bf16* __restrict__ out,
                                                        int transposed, unsigned* __restrict__ ticket) {
  if (ticket && blockIdx.x == 0 && threadIdx.x == 0) *ticket = 0;
  constexpr int FRAG = frag(D), PIECES = FRAG / 8;
  const int per = transposed ? 2 * PIECES : PIECES, i = blockIdx.x * 256 + threadIdx.x;   // a whole number of workgroups
  const int h = i / per, r = i - h * per, l = r & 63;
  V += (size_t)h * FRAG_MH * D;
  U += (size_t)h * FRAG_MH * D;
  float v[8];
  if (r < PIECES) {
    const int q = r >> 6, m = q & 1, ks = (q >> 1) % (D / 16), w = (q >> 1) / (D / 16);
    const float* src = (m ? U : V) + (size_t)(32 * w + (l & 31)) * D + ks * 16 + (l >> 5) * 8;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = src[e];
  } else {
    const int q = (r - PIECES) >> 6, ks = q % (2 * FRAG_MH / 16), b = q / (2 * FRAG_MH / 16);
    const int u = ks * 16 + (l >> 5) * 8, d = 32 * b + (l & 31);
    const float* src = (u < FRAG_MH ? V + (size_t)u * D : U + (size_t)(u - FRAG_MH) * D) + d;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = src[(size_t)e * D];
  }
  bf16x8 t;
#pragma unroll
  for (int e = 0; e < 8; ++e) t[e] = (bf16)v[e];
  *reinterpret_cast<bf16x8*>(out + (size_t)h * 2 * FRAG + (size_t)r * 8) = t;
}

constexpr int RB = 32;   // rows per block

// D = 768: [V;U] is 384 KB per 128 gate units and streams from L2 for every block of 32 rows, four times the block's own bytes as
// bf16 and as many clocks of a unit's L1 as the block needs of its share of HBM.  So nothing else may be in the way: the fragments go
// from L2 into registers in their own order (no LDS, no barriers along K), requested four slices ahead and across the blocks'
// ends, and a workgroup's serial parts (its rows' trip from memory, the gates, the softmax terms) are hidden by a second workgroup on the
// unit: the rows are in registers as fp32 for the weighted sum, only their bf16 image is in LDS.  (Weights through an LDS ring with a barrier
// per 32 columns, rows as fp32 in LDS, one workgroup per unit: 45,056 rows, M_h = 128 99 us, this
// way 47 (2.9 TB/s of rows); serving 65,536 rows 129 / 69 us, M_h = 256 264 / 98, 1,037 rows 27 / 19.)
template <int NH>   // sets of 128 gate units
__global__ void __launch_bounds__(256, 2) pool_gate_part_stream_k(PoolArgs p, const bf16* __restrict__ VU) {
  constexpr int D = 768, LDB = D + 8, KS = D / 16, CJ = D / 128, NR = 4 * CJ, PF = 4, MH = NH * FRAG_MH;
  static_assert(KS % PF == 0 && PF % 2 == 0, "rings");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16* Hb = reinterpret_cast<bf16*>(smem);                            // [RB][LDB]
  float* gb = reinterpret_cast<float*>(Hb + RB * LDB);                 // bV[MH], bU[MH], w[MH]
  float* apart = gb + 3 * MH;                                          // [4][RB]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 31, h2 = lane >> 5;
  const int rgrp = tid >> 5, cl = tid & 31;   // a thread's rows 4 rgrp .. + 3 of a block, column groups cl + 32 j
  const long long groups = (p.N + RB - 1) / RB;
  for (int j = tid; j < MH; j += 256) { gb[j] = p.Vb[j]; gb[MH + j] = p.Ub[j]; gb[2 * MH + j] = p.w[j]; }

  float4 rs[NR];
  auto load_rows = [&](long long g) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      long long row = g * RB + 4 * rgrp + k;   // rows past the end re-read the last one (their softmax term is zero)
      if (row > p.N - 1) row = p.N - 1;
      const float* h = p.H + row * D + cl * 4;
#pragma unroll
      for (int j = 0; j < CJ; ++j) rs[k * CJ + j] = *reinterpret_cast<const float4*>(h + j * 128);
    }
  };
  // fragments: set hf, this wavefront's 32 units, slice ks, V then U
  const u32x4* wr = reinterpret_cast<const u32x4*>(VU) + (size_t)wave * KS * 2 * 64 + lane;
  constexpr int SET = 2 * frag(D) / 8;   // pieces from one set to the next (the room is laid out for transposes behind each)
  u32x4 wf[PF][2];
  int opaque = 0;   // written anew for every block: the same fragments are not to be kept in registers from one to the next
  auto load_w = [&](int slot, int hf, int ks) __attribute__((always_inline)) {
    const u32x4* q = wr + opaque + hf * SET + ks * 128;
    wf[slot][0] = q[0];
    wf[slot][1] = q[64];
  };
  double z[4 * CJ];   // the weighted sum feeds a cancelling difference in the backward
#pragma unroll
  for (int i = 0; i < 4 * CJ; ++i) z[i] = 0.0;
  float run_m = -INFINITY;
  double lsum = 0.0;

  load_rows(blockIdx.x);
#pragma unroll
  for (int i = 0; i < PF; ++i) load_w(i, 0, i);
  const bf16* hrow = Hb + li * LDB + h2 * 8;
  for (long long g = blockIdx.x; g < groups; g += gridDim.x) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int j = 0; j < CJ; ++j) {
        const float4 v = rs[k * CJ + j];
        f32x2 p0 = {v.x, v.y}, p1 = {v.z, v.w};
        uint2 w2;
        w2.x = __builtin_bit_cast(unsigned, __builtin_convertvector(p0, bf16x2));
        w2.y = __builtin_bit_cast(unsigned, __builtin_convertvector(p1, bf16x2));
        *reinterpret_cast<uint2*>(Hb + (4 * rgrp + k) * LDB + (cl + 32 * j) * 4) = w2;
      }
    asm volatile("" : "+s"(opaque));
    step_barrier();   // the image is visible, the last block's partial logits are read (loads stay in flight)
    float part = 0.f;
#pragma unroll 1
    for (int hf = 0; hf < NH; ++hf) {
      f32x16 av, au;
#pragma unroll
      for (int r = 0; r < 16; ++r) av[r] = au[r] = 0.f;
      u32x4 hb[2];
      hb[0] = *reinterpret_cast<const u32x4*>(hrow);
      static_for<0, KS>([&](auto kc) __attribute__((always_inline)) {
        constexpr int ks = decltype(kc)::value, sl = ks % PF;
        if constexpr (ks + 1 < KS) hb[(ks + 1) % 2] = *reinterpret_cast<const u32x4*>(hrow + (ks + 1) * 16);
        const bf16x8 f = __builtin_bit_cast(bf16x8, hb[ks % 2]);
        av = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wf[sl][0]), f, av, 0, 0, 0);
        au = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wf[sl][1]), f, au, 0, 0, 0);
        if constexpr (ks + PF < KS) load_w(sl, hf, ks + PF);
        else load_w(sl, hf + 1 < NH ? hf + 1 : 0, ks + PF - KS);   // the next set's, or the next block's
        __builtin_amdgcn_sched_barrier(0);
      });
      // accumulator register r of a lane = gate unit (r / 4) * 8 + h2 * 4 + r % 4 of the wavefront's 32, row li
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = hf * FRAG_MH + wave * 32 + q * 8 + h2 * 4;
        const float4 bv = *reinterpret_cast<const float4*>(gb + j), bu = *reinterpret_cast<const float4*>(gb + MH + j);
        const float4 wj = *reinterpret_cast<const float4*>(gb + 2 * MH + j);
        const float bvv[4] = {bv.x, bv.y, bv.z, bv.w}, buu[4] = {bu.x, bu.y, bu.z, bu.w}, ww[4] = {wj.x, wj.y, wj.z, wj.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float xv = av[4 * q + e] + bvv[e], xu = au[4 * q + e] + buu[e];
          // tanh(xv) * sigmoid(xu) = (1 - e1) / ((1 + e1) (1 + e2)), e1 = exp(-2 xv), e2 = exp(-xu)
          const float e1 = __expf(fminf(-2.0f * xv, 40.f)), e2 = __expf(fminf(-xu, 40.f));
          part += ww[e] * ((1.0f - e1) * __builtin_amdgcn_rcpf((1.0f + e1) * (1.0f + e2)));
        }
      }
    }
    part += __shfl_xor(part, 32, 64);
    if (h2 == 0) apart[wave * RB + li] = part;
    step_barrier();   // the four partial logits of every row are there, the image is free
    // softmax terms, by every wavefront for itself: lanes li and li + 32 have row li
    const long long n0 = g * RB;
    const bool ok = n0 + li < p.N;
    float a = apart[li] + apart[RB + li] + apart[2 * RB + li] + apart[3 * RB + li];
    if (wave == 0 && h2 == 0 && ok) p.a[n0 + li] = a;
    a = ok ? a : -INFINITY;
    const float m = fmaxf(run_m, wave_max(a));   // finite: the block has at least one row
    const float e = __expf(a - m);
    const double sc = (double)__expf(run_m - m);   // exp(-inf) = 0 on the first block
    run_m = m;
    lsum = lsum * sc + (double)e;   // summed over the rows once, at the end
    double ek[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) ek[k] = (double)__shfl(e, 4 * (rgrp & 7) + k, 64);
#pragma unroll
    for (int j = 0; j < CJ; ++j) {
      double s[4] = {z[4 * j] * sc, z[4 * j + 1] * sc, z[4 * j + 2] * sc, z[4 * j + 3] * sc};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float4 v = rs[k * CJ + j];
        s[0] += ek[k] * (double)v.x; s[1] += ek[k] * (double)v.y; s[2] += ek[k] * (double)v.z; s[3] += ek[k] * (double)v.w;
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) z[4 * j + c] = s[c];
    }
    __builtin_amdgcn_sched_barrier(0);
    if (g + gridDim.x < groups) load_rows(g + gridDim.x);   // uniform
  }
  // column sums over the 8 row groups (every wavefront is past the last barrier, so the image is dead)
  double* zred = reinterpret_cast<double*>(smem);   // [8][D]
  static_assert(8 * D * 8 <= RB * LDB * 2, "reduction buffer");
#pragma unroll
  for (int j = 0; j < CJ; ++j)
#pragma unroll
    for (int c = 0; c < 4; ++c) zred[rgrp * D + (cl + 32 * j) * 4 + c] = z[4 * j + c];
  __syncthreads();
  double* out = p.part + (size_t)blockIdx.x * (2 + D);
  for (int o = 1; o < 32; o <<= 1) lsum += __shfl_xor(lsum, o, 64);   // one half has all rows
  if (tid == 0) { out[0] = (double)run_m; out[1] = lsum; }
  for (int d = tid; d < D; d += 256) {
    double t = 0.0;
#pragma unroll
    for (int g = 0; g < 8; ++g) t += zred[g * D + d];
    out[2 + d] = t;
  }
}

// Variant for the shape whose [V;U] fits the register file (D = 384, M_h = 128: 2 M_h * D bf16 = 192 KB, 192
// registers per lane): each wavefront holds the MFMA fragments of its 32 gate units for the whole kernel, so the only
// traffic per block of 32 feature rows is the block itself (the kernel above re-reads the weights from L2 for every
// block, four times the bytes of the features).
//   * A thread owns 4 rows x 12 columns of every block (fixed columns), in fp32 registers.  LDS holds only the bf16
//     image of a block (double buffered) for the MFMA fragments; the weighted feature sum is taken from the fp32
//     registers: per lane in fp32 (4 rows per block: one term per 2,048 rows of the bag, 64 at 131,072 rows), over row groups and
//     workgroups in fp64 (z feeds a cancelling difference in the backward).
//   * The gate of block i - 1 runs under the MFMAs of block i inside each wavefront (the matrix pipe and the vector
//     ALU are separate, and with one wavefront per SIMD nothing else overlaps them).  The pre-activations of two
//     blocks are alive (two accumulator sets), and the softmax terms, hence the weighted sum, of a block come one
//     iteration after its MFMAs: three fp32 row sets rotate (block i - 1 waiting for its weights, block i whose bf16
//     image is being multiplied, block i + 1 in flight).  The set that the weighted sum frees takes the first loads
//     of block i + 2 at once.  The roles repeat every 6 iterations (2 images x 3 row sets), which are written out.
//   * Every wavefront computes the block's softmax terms itself from the four partial logits (no serial section).
//   * Two barriers per block: partial logits visible; next bf16 image visible.
//   * NH = 2: two such sets of gate units one after the other, each a pass over the workgroup's blocks: the first leaves its partial
//     logits in a_tmp, the second adds them and does everything else.  A launch for each paid for ramp and drain twice:
//     45,056 rows, two of a training step 77 us, this way 74 (a step 223 -> 219).
constexpr int POOL_REG_NL = 4;   // weight slices read from LDS (the rest stay in registers)
template <int D, int MH, int NH>
__global__ void __launch_bounds__(256) pool_gate_part_reg_k(PoolArgs p, const bf16* __restrict__ VU) {
  constexpr int LDB = D + 8, KS = D / 16, CJ = D / 128, NR = 4 * CJ, EARLY = CJ;
  constexpr int NL = POOL_REG_NL, KR = KS - NL;   // the last NL slices of the weights are read from LDS
  static_assert(MH == 128 && D % 128 == 0 && KS % 3 == 0 && KS / 3 * 2 == 16 && NR - EARLY <= KS && EARLY % CJ == 0, "shape");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16* Hb = reinterpret_cast<bf16*>(smem);                            // [2][RB][LDB]
  u32x4* Wl = reinterpret_cast<u32x4*>(Hb + 2 * RB * LDB);             // [4 waves][NL][2][64 lanes] weight fragments
  float* gb = reinterpret_cast<float*>(Wl + 4 * NL * 2 * 64);          // scaled bV[MH], scaled bU[MH], w[MH]
  float* apart = gb + 3 * MH;                                          // [4][RB]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 31, h2 = lane >> 5;
  const int rgrp = tid >> 5, cl = tid & 31;   // loads: rows 4 rgrp .. + 3 of a block, column groups cl + 32 j
  const float* H = p.H;
  const long long groups = (p.N + RB - 1) / RB;
  constexpr float C1 = -2.0f * 1.44269504088896f, C2 = -1.44269504088896f;   // exp(-2x) and exp(-x) as exp2
  constexpr int FRAG = frag(D);
  if (const int hf = blockIdx.y) {   // the second half of the gate units beside the first
    VU += (size_t)hf * 2 * FRAG;
    p.Vb += hf * MH; p.Ub += hf * MH; p.w += hf * MH;
    p.a += hf * p.N;
  }

  auto fill_gb = [&](int pass) __attribute__((always_inline)) {
    for (int j = tid; j < MH; j += 256) { gb[j] = C1 * p.Vb[pass * MH + j]; gb[MH + j] = C2 * p.Ub[pass * MH + j]; gb[2 * MH + j] = p.w[pass * MH + j]; }
  };
  if constexpr (NH == 1) fill_gb(0);   // (behind the sums of |w|, serving 65,536 rows took 33.3 us instead of 32.3)

  // this wavefront's gate units 32 wave .. + 31 of V and of U: slices 0 .. KR - 1 of their weights stay in the
  // accumulation half of the register file (the MFMA reads them there), the last NL go to LDS in fragment order
  // (each lane reads back what it wrote): with all of them in registers the two accumulator sets fill that half
  // to the last register and the allocator spills
  bf16x8 wv[KR], wu[KR];
  u32x4* wl = Wl + (size_t)wave * NL * 2 * 64 + lane;
  float4 rs[3][NR];
  f32x16 acc[2][2];
  // The blocks of a workgroup are loaded strictly one after the other (load 0 .. NR - 1 of a block, then the next
  // block), so one running row index serves every load site; 32-bit (N < 2^31 - 2^24 is checked on the host).
  const unsigned lastrow = (unsigned)(p.N - 1), lstep = gridDim.x * RB;
  unsigned lrow = blockIdx.x * RB + 4 * rgrp;   // first of this thread's 4 rows of the block being loaded
  const float* hrp = H;                         // row base of the loads in progress
  // load i = k * CJ + j; rows past the end re-read the last row (their softmax term is set to zero)
  auto issue_one = [&](float4 (&r)[NR], auto ic) __attribute__((always_inline)) {
    constexpr int i = decltype(ic)::value, k = i / CJ, j = i % CJ;
    if constexpr (j == 0) {
      unsigned row = lrow + k;
      row = row < lastrow ? row : lastrow;
      hrp = H + (size_t)row * D + cl * 4;
    }
    r[i] = *reinterpret_cast<const float4*>(hrp + j * 128);
    if constexpr (i == NR - 1) lrow += lstep;
  };
  auto stash_one = [&](const float4 (&r)[NR], int buf, auto ic) __attribute__((always_inline)) {
    constexpr int i = decltype(ic)::value, k = i / CJ, j = i % CJ;
    float4 v = r[i];
    f32x2 p0 = {v.x, v.y}, p1 = {v.z, v.w};
    bf16x2 h0 = __builtin_convertvector(p0, bf16x2), h1 = __builtin_convertvector(p1, bf16x2);
    uint2 w2;
    w2.x = __builtin_bit_cast(unsigned, h0);
    w2.y = __builtin_bit_cast(unsigned, h1);
    *reinterpret_cast<uint2*>(Hb + (buf * RB + 4 * rgrp + k) * LDB + (cl + 32 * j) * 4) = w2;
  };
  auto stash_h = [&](const float4 (&r)[NR], int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int j = 0; j < CJ; ++j) {
        float4 v = r[k * CJ + j];
        f32x2 p0 = {v.x, v.y}, p1 = {v.z, v.w};
        bf16x2 h0 = __builtin_convertvector(p0, bf16x2), h1 = __builtin_convertvector(p1, bf16x2);
        uint2 w2;
        w2.x = __builtin_bit_cast(unsigned, h0);
        w2.y = __builtin_bit_cast(unsigned, h1);
        *reinterpret_cast<uint2*>(Hb + (buf * RB + 4 * rgrp + k) * LDB + (cl + 32 * j) * 4) = w2;
      }
  };
  // fp32 partial sums: a lane adds 4 rows per block, N / 2048 terms in all (256 workgroups x 8 row groups), before the fp64 reduction over row
  // groups and workgroups
  float z[4 * CJ];
  float wabs = 0.f;
  for (int j = lane; j < NH * MH; j += 64) wabs += fabsf(p.w[j]);
  wabs = wave_sum(wabs);
  const bool fixed = wabs <= 40.f;   // a bound of every logit serves as the softmax shift
  float run_m = fixed ? wabs : -INFINITY;
  double lsum = 0.0;
  if constexpr (NH == 1) {
#pragma unroll
    for (int i = 0; i < 4 * CJ; ++i) z[i] = 0.f;
  }
  const int st = gridDim.x;
  const int nblk = (int)((groups - blockIdx.x + st - 1) / st);   // blocks of this workgroup (>= 1)
  int pass = 0;

  // iteration `it` (role phase ph = it mod 6): MFMAs of block it (on the last image again when it == nblk: unused),
  // gate, softmax terms and weighted sum of block it - 1, loads of block it + 1 (and the first of block it + 2)
  auto iter = [&](auto phc, int it) __attribute__((always_inline)) {
    constexpr int ph = decltype(phc)::value, buf = ph & 1, ls = (ph + 1) % 3, zs = (ph + 2) % 3;
    f32x16 (&ac)[2] = acc[ph & 1];
    const f32x16 (&ap)[2] = acc[(ph & 1) ^ 1];
#pragma unroll
    for (int r = 0; r < 16; ++r) { ac[0][r] = 0.f; ac[1][r] = 0.f; }
    const bf16* hrow = Hb + (buf * RB + li) * LDB + h2 * 8;
    constexpr int PF = 3;
    u32x4 hf[PF];
#pragma unroll
    for (int ks = 0; ks < PF; ++ks) hf[ks] = *reinterpret_cast<const u32x4*>(hrow + ks * 16);
    float part = 0.f, part2 = 0.f;
    u32x4 lw[2][2];
    const float* gbl = gb + 32 * wave + h2 * 4;   // scaled biases and w of this lane's gate units
    float2 bv2 = *reinterpret_cast<const float2*>(gbl), bu2, w2;
    float ge1[2], ge2[2], gnum[2];
    // Gate of the previous block, two elements (accumulator registers 2t, 2t + 1) at a time in three stages, one per
    // slice, a new pair every second slice (slices 2t, 2t + 1, 2t + 2): the vector ALU always has independent chains
    // and a slice's share stays under the 64 clocks of its two MFMAs.  Accumulator register r of a lane = gate unit
    // (r / 4) * 8 + h2 * 4 + r % 4 of the wavefront's 32, row li.  The finished accumulators are read where they are,
    // in the accumulation half of the register file (left to itself the allocator moves them to 32 ordinary registers
    // first, which the three row sets need).
    // tanh(xv) * sigmoid(xu) = (1 - e1) / ((1 + e1) (1 + e2)), e1 = exp(-2 xv), e2 = exp(-xu)
    auto gate0 = [&](auto tc) __attribute__((always_inline)) {
      constexpr int t = decltype(tc)::value, r0 = 2 * t, off = (r0 / 4) * 8 + r0 % 4;
      bu2 = *reinterpret_cast<const float2*>(gbl + MH + off);
      w2 = *reinterpret_cast<const float2*>(gbl + 2 * MH + off);
      float xa, xb;
      asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(xa) : "a"(ap[0][r0]));
      asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(xb) : "a"(ap[0][r0 + 1]));
      ge1[0] = __builtin_amdgcn_exp2f(fminf(fmaf(xa, C1, bv2.x), 57.f));
      ge1[1] = __builtin_amdgcn_exp2f(fminf(fmaf(xb, C1, bv2.y), 57.f));
    };
    auto gate1 = [&](auto tc) __attribute__((always_inline)) {
      constexpr int t = decltype(tc)::value, r0 = 2 * t;
      float xa, xb;
      asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(xa) : "a"(ap[1][r0]));
      asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(xb) : "a"(ap[1][r0 + 1]));
      ge2[0] = __builtin_amdgcn_exp2f(fmaf(xa, C2, bu2.x));   // inf is fine: 1 / inf = 0, e1 is finite
      ge2[1] = __builtin_amdgcn_exp2f(fmaf(xb, C2, bu2.y));
      gnum[0] = fmaf(-w2.x, ge1[0], w2.x);
      gnum[1] = fmaf(-w2.y, ge1[1], w2.y);
      ge1[0] = fmaf(ge1[0] + 1.0f, ge2[0], ge1[0] + 1.0f);   // (1 + e1) (1 + e2)
      ge1[1] = fmaf(ge1[1] + 1.0f, ge2[1], ge1[1] + 1.0f);
      if constexpr (t + 1 < 8) {   // the next pair's first constants
        constexpr int r1 = r0 + 2, off1 = (r1 / 4) * 8 + r1 % 4;
        bv2 = *reinterpret_cast<const float2*>(gbl + off1);
      }
    };
    float gden[2];
    auto gate2 = [&]() __attribute__((always_inline)) {
      part = fmaf(gnum[0], __builtin_amdgcn_rcpf(gden[0]), part);
      part2 = fmaf(gnum[1], __builtin_amdgcn_rcpf(gden[1]), part2);
    };
    // After the last gate stage (slice GA): the partial logits are exchanged, and the softmax terms, the weighted sum
    // of block it - 1, the first loads of block it + 2 and the bf16 image of block it + 1 run under the remaining
    // slices' MFMAs.
    constexpr int GA = 16, SP = (KS - 1 - GA - CJ);   // SP slices share the NR registers of the image
    static_assert(GA + CJ + 1 < KS && NR % SP == 0, "tail schedule");
    const long long n0 = ((long long)blockIdx.x + (long long)(it - 1) * st) * RB;   // first row of block it - 1
    float a_out = 0.f, sc = 1.0f, ek[4] = {0.f, 0.f, 0.f, 0.f};
    float a_prev = 0.f;   // the first pass's partial logit of this lane's row
    if (NH > 1 && pass > 0 && it >= 1) a_prev = p.a_tmp[n0 + li < p.N ? n0 + li : p.N - 1];   // uniform
    static_for<0, KS>([&](auto kc) __attribute__((always_inline)) {
      constexpr int ks = decltype(kc)::value;
      bf16x8 f = __builtin_bit_cast(bf16x8, hf[ks % PF]);
      if constexpr (ks + PF < KS) hf[ks % PF] = *reinterpret_cast<const u32x4*>(hrow + (ks + PF) * 16);
      // one load per slice: issued as one burst they hold the wavefronts in the issue for the ~770 clocks the address
      // unit needs for a block's 48 KB
      if constexpr (ks + EARLY < NR) issue_one(rs[ls], IC<ks + EARLY>{});
      if constexpr (ks < KR) {
        ac[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wv[ks], f, ac[0], 0, 0, 0);
        ac[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wu[ks], f, ac[1], 0, 0, 0);
      } else {
        ac[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, lw[(ks - KR) % 2][0]), f, ac[0], 0, 0, 0);
        ac[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, lw[(ks - KR) % 2][1]), f, ac[1], 0, 0, 0);
      }
      if constexpr (ks + 2 >= KR && ks + 2 < KS) {   // weight fragments from LDS, two slices ahead
        lw[(ks + 2 - KR) % 2][0] = wl[((ks + 2 - KR) * 2 + 0) * 64];
        lw[(ks + 2 - KR) % 2][1] = wl[((ks + 2 - KR) * 2 + 1) * 64];
      }
      if constexpr (ks % 2 == 0 && ks >= 2 && ks <= GA) gate2();                      // pair (ks - 2) / 2
      if constexpr (ks % 2 == 0 && ks / 2 < 8) gate0(IC<ks / 2>{});
      if constexpr (ks % 2 == 1 && ks / 2 < 8) { gate1(IC<ks / 2>{}); gden[0] = ge1[0]; gden[1] = ge1[1]; }
      if constexpr (ks == GA) {
        part += part2;
        part += __shfl_xor(part, 32, 64);
        if (h2 == 0) apart[wave * RB + li] = part;
        __syncthreads();   // (A) the four partial logits of every row of block it - 1 are there
        if (it >= 1) {     // uniform
          float a = apart[li] + apart[RB + li] + apart[2 * RB + li] + apart[3 * RB + li] + a_prev;
          const bool ok = n0 + li < p.N;
          a_out = a;
          float e;
          if (NH > 1 ? pass + 1 < NH : p.partial != 0) {   // uniform: only the partial logits are wanted
            e = 0.f;
          } else if (fixed) {   // uniform
            e = ok ? __expf(a - run_m) : 0.f;
          } else {
            a = ok ? a : -INFINITY;
            float m = fmaxf(run_m, wave_max(a));   // finite: the block has at least one row
            e = __expf(a - m);                     // lanes li and li + 32: row li
            sc = __expf(run_m - m);                // exp(-inf) = 0 on the first block
            run_m = m;
            lsum *= (double)sc;
          }
          lsum += (double)e;   // summed over the rows once, at the end
#pragma unroll
          for (int k = 0; k < 4; ++k) ek[k] = __shfl(e, 4 * (rgrp & 7) + k, 64);
        }
      }
      if constexpr (ks > GA && ks <= GA + CJ) {   // weighted sum, one group of 4 columns per slice (all zero when it = 0)
        constexpr int j = ks - GA - 1;
        float4 s = make_float4(z[4 * j] * sc, z[4 * j + 1] * sc, z[4 * j + 2] * sc, z[4 * j + 3] * sc);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          float4 v = rs[zs][k * CJ + j];
          s.x = fmaf(ek[k], v.x, s.x); s.y = fmaf(ek[k], v.y, s.y);
          s.z = fmaf(ek[k], v.z, s.z); s.w = fmaf(ek[k], v.w, s.w);
        }
        z[4 * j] = s.x; z[4 * j + 1] = s.y; z[4 * j + 2] = s.z; z[4 * j + 3] = s.w;
      }
      if constexpr (ks == GA + CJ) {
        // the freed set takes the first loads of block it + 2 (the next iteration continues with load EARLY); they
        // must not move above the weighted sum, which still reads the registers they land in
        asm volatile("" ::: "memory");
        static_for<0, EARLY>([&](auto ic) __attribute__((always_inline)) { issue_one(rs[zs], ic); });
      }
      if constexpr (ks > GA + CJ) {   // bf16 image of block it + 1 (replaces that of block it - 1), NR / SP registers per slice
        constexpr int q = ks - GA - CJ - 1;
        static_for<q * (NR / SP), (q + 1) * (NR / SP)>([&](auto ic) __attribute__((always_inline)) { stash_one(rs[ls], buf ^ 1, ic); });
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    // both accumulator sets stay in the accumulation half of the register file (left to itself the allocator moves
    // the finished one to 32 ordinary registers, which the three row sets need)
    asm volatile("" : "+a"(ac[0]), "+a"(ac[1]));
    if (it >= 1 && wave == 0 && h2 == 0 && n0 + li < p.N) (pass + 1 < NH ? p.a_tmp : p.a)[n0 + li] = a_out;   // kept for the backward
    __syncthreads();   // (B) the next bf16 image is visible; apart is free again
  };

  for (;; ++pass) {
    // prologue: block 0 of this workgroup, and the first loads of block 1 (every wavefront is past the last barrier (B) of the pass before)
    if constexpr (NH > 1) {
      lrow = blockIdx.x * RB + 4 * rgrp;
#pragma unroll
      for (int i = 0; i < 4 * CJ; ++i) z[i] = 0.f;
    }
    if constexpr (NH > 1) fill_gb(pass);
    static_for<0, NR>([&](auto ic) __attribute__((always_inline)) { issue_one(rs[0], ic); });
    static_for<0, EARLY>([&](auto ic) __attribute__((always_inline)) { issue_one(rs[1], ic); });
    // the weights, while the rows come from memory; all of them are requested before the first is waited for (one at a time, each
    // a trip to L2, 1,037 rows take 11.7 us instead of 8.9 and 45,056 rows 22.3 instead of 19.2)
    {
      const u32x4* wr = reinterpret_cast<const u32x4*>(VU + (size_t)pass * 2 * FRAG) + (size_t)wave * KS * 2 * 64 + lane;   // fragment order
      u32x4 a[2 * KS];
#pragma unroll
      for (int i = 0; i < 2 * KS; ++i) a[i] = wr[i * 64];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (ks < KR) {
          asm volatile("" : "+a"(a[2 * ks]), "+a"(a[2 * ks + 1]));
          wv[ks] = __builtin_bit_cast(bf16x8, a[2 * ks]);
          wu[ks] = __builtin_bit_cast(bf16x8, a[2 * ks + 1]);
        } else {
          wl[((ks - KR) * 2 + 0) * 64] = a[2 * ks];
          wl[((ks - KR) * 2 + 1) * 64] = a[2 * ks + 1];
        }
      }
    }
    stash_h(rs[0], 0);
    // iteration 0 has no previous block: its gate reads zeros and its weighted sum adds zero times zero
#pragma unroll
    for (int i = 0; i < NR; ++i) rs[2][i] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int r = 0; r < 16; ++r) { acc[1][0][r] = 0.f; acc[1][1][r] = 0.f; }
    __syncthreads();
    for (int it = 0;;) {
      iter(IC<0>{}, it); if (++it > nblk) break;
      iter(IC<1>{}, it); if (++it > nblk) break;
      iter(IC<2>{}, it); if (++it > nblk) break;
      iter(IC<3>{}, it); if (++it > nblk) break;
      iter(IC<4>{}, it); if (++it > nblk) break;
      iter(IC<5>{}, it); if (++it > nblk) break;
    }
    if (pass + 1 == NH) break;
  }
  if (p.partial) return;
  // column sums over the 8 row groups (the bf16 images are dead: every wavefront is past the last barrier (B))
  double* zred = reinterpret_cast<double*>(smem);   // [8][D]
  static_assert(8 * D * 8 <= 2 * RB * LDB * 2, "reduction buffer");
#pragma unroll
  for (int j = 0; j < CJ; ++j)
#pragma unroll
    for (int c = 0; c < 4; ++c) zred[rgrp * D + (cl + 32 * j) * 4 + c] = (double)z[4 * j + c];
  __syncthreads();
  double* out = p.part + (size_t)blockIdx.x * (2 + D);
  // lanes li and li + 32 hold the same rows: sum over one half
  for (int o = 1; o < 32; o <<= 1) lsum += __shfl_xor(lsum, o, 64);
  if (tid == 0) { out[0] = (double)run_m; out[1] = lsum; }
  for (int d = tid; d < D; d += 256) {
    double t = 0.0;
#pragma unroll
    for (int g = 0; g < 8; ++g) t += zred[g * D + d];
    out[2 + d] = t;
  }
}

// NH passes in a workgroup, or `halves` sets of gate units side by side
template <int NH>
hipError_t go_reg(const PoolArgs& p, const bf16* vu, hipStream_t s, int halves = 1) {
  constexpr int D = FRAG_D, MH = FRAG_MH;
  auto kern = pool_gate_part_reg_k<D, MH, NH>;
  size_t lds = (size_t)2 * 32 * (D + 8) * 2 + (size_t)4 * POOL_REG_NL * 2 * 64 * 16 + (size_t)3 * MH * 4 + 4 * 32 * 4;
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(p.blocks, halves), dim3(256), lds, s, p, vu);
  return hipGetLastError();
}

// M_h = 256.  Below 32,768 rows both halves of the gate units run side by side, 128 workgroups each, and leave their partial logits; the
// softmax partials are a launch of their own, with the largest logit as the shift and the weighted sum in float64.  From there on both
// halves are passes of one launch over the rows, with the logits' bound as the shift and a lane's sums in float32: faster, but the softmax weights
// are off by 1.3e-7 instead of 0.4e-7 (operands on the bf16 grid, against 64 bits), so it does not go below the line from which on it has
// always been so.  us, side by side / one launch: serving 1,037 rows 21.5 / 29.6, 4,096 22.7 / 24.6, 8,192 26.2 / 25.6, 16,384 33.5 / 29.0,
// 32,000 45.5 / 40.2; training step 16,384 141 / 130, 32,000 192 / 178.  (With the weights streaming from L2 for every block of rows:
// serving 16,384 rows 36.1, 32,000 63; training 166 and 253.)
constexpr long long SIDE_BY_SIDE_ROWS = 32768;
hipError_t go_reg_halves(PoolArgs& p0, hipStream_t s) {
  PoolArgs p = p0;
  p.Mh = FRAG_MH;
  if (p.N < SIDE_BY_SIDE_ROWS && (size_t)p.N * 2 <= p.a_room) {
    p.partial = 1;
    if (p.blocks > 128) p.blocks = 128;   // half of the chip each
    p.a = p0.a_tmp;
    hipError_t e = go_reg<1>(p, (const bf16*)p0.vub, s, 2);
    if (e != hipSuccess) return e;
    p0.blocks = pool_blocks(p0.N);
    return launch_pool_softmax_part(p0, p0.a_tmp, 2, s);
  }
  return go_reg<2>(p, (const bf16*)p0.vub, s);
}

template <int NH>
hipError_t go_stream(PoolArgs& p, hipStream_t s) {
  auto kern = pool_gate_part_stream_k<NH>;
  const size_t lds = (size_t)RB * (768 + 8) * 2 + (size_t)3 * NH * FRAG_MH * 4 + 4 * RB * 4;
  const long long groups = (p.N + RB - 1) / RB;   // two workgroups per compute unit
  p.blocks = groups < 2 * p.blocks ? (int)groups : 2 * p.blocks;
  if (p.blocks > 1024) p.blocks = 1024;
  hipLaunchKernelGGL(kern, dim3(p.blocks), dim3(256), lds, s, p, (const bf16*)p.vub);
  return hipGetLastError();
}

}  // namespace

// shapes built: (D, M_h) in {384, 768} x {128, 256}
bool pool_mfma_ok(const PoolArgs& p) {
  return p.vub && p.N >= 512 && p.N < (1LL << 31) - (1 << 24) && (p.D == 384 || p.D == 768) && (p.Mh == 128 || p.Mh == 256) &&
         ((uintptr_t)p.H & 15) == 0 && ((uintptr_t)p.vub & 15) == 0;
}

// whether the forward leaves the weights in fragment order in p.vub (with their transposes if p.G is set)
bool pool_frag_fwd(const PoolArgs& p) {
  return p.use_mfma && pool_mfma_ok(p) && p.D == FRAG_D;
}

hipError_t launch_pool_cast_frag(const PoolArgs& p, bool transposed, unsigned* ticket, hipStream_t s) {
  const int pieces = p.Mh / FRAG_MH * (frag(p.D) / 8) * (transposed ? 2 : 1);
  auto kern = p.D == FRAG_D ? pool_cast_frag_k<FRAG_D> : pool_cast_frag_k<768>;
  hipLaunchKernelGGL(kern, dim3(pieces / 256), dim3(256), 0, s, p.VW, p.UW, (bf16*)p.vub, (int)transposed, ticket);
  return hipGetLastError();
}

hipError_t launch_pool_gate_part_mfma(PoolArgs& p, hipStream_t s) {
  const bool narrow = pool_frag_fwd(p);
  hipError_t e = launch_pool_cast_frag(p, narrow && p.G != nullptr, p.ticket, s);
  if (e != hipSuccess) return e;
  if (narrow) return p.Mh == FRAG_MH ? go_reg<1>(p, (const bf16*)p.vub, s) : go_reg_halves(p, s);
  return p.Mh == FRAG_MH ? go_stream<1>(p, s) : go_stream<2>(p, s);
}

}  // namespace sl
