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

// Eight floats as three bf16 vectors whose sum they are, bit for bit, from 2^-110 in size on (a trailing term ends at 2^-133).  Each term is
// the rest rounded to nearest, so that the next one is at most half a unit of its last place and has either sign.  (A float that rounds up to
// an infinite leading term has no trailing ones: not_finite.)
// `up` is 1, or +-2^48 with which the vectors are exact for every float.  So go a product's first operands, where gradients are: those of a
// tile that the attention has all but left out may be as small as floats get, while weights and activations are not.  The results are
// scaled back (scale_down); operands of 2^80 and results as large are infinite on the way, and those blocks are taken again.
struct Split { bf16x8 t[3]; };   // leading, middle, trailing bits
constexpr float SPLIT_UP = 0x1p48f;
__host__ __device__ __forceinline__ Split split8(const float (&x)[8], float up = 1.f) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  u32x4 w[3];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    f32x2 v = {x[2 * p] * up, x[2 * p + 1] * up};
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      w[i][p] = __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
      v[0] -= __builtin_bit_cast(float, w[i][p] << 16);
      v[1] -= __builtin_bit_cast(float, w[i][p] & 0xffff0000u);
    }
  }
  Split s;
#pragma unroll
  for (int i = 0; i < 3; ++i) s.t[i] = __builtin_bit_cast(bf16x8, w[i]);
  return s;
}
__device__ __forceinline__ Split split_of(f32x4 a, f32x4 b, float up = 1.f) {
  return split8({a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]}, up);
}
// The matrix core adds a step's products with a slight pull downwards (results are 2e-8 to 2e-7 of their mean size low), which the float32
// form has not.  Where a result is the sum of several wavefronts' or slabs' parts, every other one takes its first operand negated.
__device__ __forceinline__ float split_up(int part) { return part & 1 ? -SPLIT_UP : SPLIT_UP; }
template <int NA, int NB>
__device__ __forceinline__ void scale_down(f32x16 (&acc)[NA][NB], float up) {
  const float down = 1.0f / SPLIT_UP / SPLIT_UP * up;
#pragma unroll
  for (int i = 0; i < NA; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] *= down;
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
// the six of the nine products of terms that are taken, the smallest first: what is left out is at most 2^-24 of a product and of either sign
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
