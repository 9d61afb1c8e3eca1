// float32 operands on the bf16 matrix cores: the cut into three bf16 terms, their image in LDS and the products that are taken
// (what this gives and costs: gemm_f32.hip).
#pragma once
#include "slide_internal.h"

namespace sl {

constexpr int SPLIT_BK = 32;   // contracted elements per step

__device__ __forceinline__ void step_barrier() {
  __builtin_amdgcn_s_waitcnt(0xc07f);   // this wavefront's LDS accesses are done (its loads from memory stay in flight)
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Eight floats as three bf16 vectors whose sum they are, bit for bit: each takes the next eight significant bits (cut off, not
// rounded, so that the largest finite float stays finite).
struct Split { bf16x8 t[3]; };   // leading, middle, trailing bits
__device__ __forceinline__ Split split8(const float (&x)[8]) {
  unsigned w[3][4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    float a = x[2 * p], b = x[2 * p + 1];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const unsigned ua = __float_as_uint(a), ub = __float_as_uint(b);
      w[i][p] = __builtin_amdgcn_perm(ub, ua, 0x07060302u);   // the upper halves of b and a
      if (i < 2) {
        a -= __uint_as_float(ua & 0xffff0000u);
        b -= __uint_as_float(ub & 0xffff0000u);
      }
    }
  }
  Split s;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    s.t[i] = __builtin_bit_cast(bf16x8, u32x4{w[i][0], w[i][1], w[i][2], w[i][3]});
  }
  return s;
}
// A step's operands in LDS: 3 planes (terms) of ROWS rows of 32 bf16; the 16-byte pieces of a row are slot-permuted (piece c of row R
// in slot c ^ ((R >> 2) & 3)), so that 16-byte accesses to 16 consecutive rows fall on 64 different banks.
template <int ROWS>
__device__ __forceinline__ void put_split(bf16* s, int row, int piece, const Split& v) {
#pragma unroll
  for (int i = 0; i < 3; ++i) *reinterpret_cast<bf16x8*>(s + (i * ROWS + row) * SPLIT_BK + (piece ^ ((row >> 2) & 3)) * 8) = v.t[i];
}
template <int ROWS>
__device__ __forceinline__ Split get_split(const bf16* s, int row, int piece) {
  Split v;
#pragma unroll
  for (int i = 0; i < 3; ++i) v.t[i] = *reinterpret_cast<const bf16x8*>(s + (i * ROWS + row) * SPLIT_BK + (piece ^ ((row >> 2) & 3)) * 8);
  return v;
}
// the six of the nine products of terms that reach the 24th bit, the smallest first
constexpr int TERM_A[6] = {0, 2, 1, 0, 1, 0}, TERM_B[6] = {2, 0, 1, 1, 0, 0};
// whether a wavefront's results are anything but finite numbers: an infinite operand (whose other terms are no numbers, where the
// product of floats may be infinite) or an overflow.  Such blocks are taken again, in float32 products.
template <int NA, int NB>
__device__ __forceinline__ bool not_finite(const f32x16 (&acc)[NA][NB]) {
  float worst = 0.f;
#pragma unroll
  for (int i = 0; i < NA; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) worst = fmaf(acc[i][j][r], 0.f, worst);   // 0, or no number
  return __any(worst != worst);
}

}  // namespace sl
