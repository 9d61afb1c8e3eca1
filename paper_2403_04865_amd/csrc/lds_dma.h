// Loads from global memory straight into LDS, in their buffer form.
//   * A buffer load is no FLAT instruction: while a global_load ... lds may be pending the compiler lets no LDS read pass and
//     waits for all of them (lgkmcnt(0)) before every use; behind the buffer form it counts.
//   * 64-bit addresses per lane become one 32-bit offset beside a uniform base and a uniform offset, and rows that do not
//     exist (padding, past the end) need no row of zeros to point at: what lies outside the buffer is loaded as zeros.
// ResNet18 step of 1024 tiles with the convolutions' loads in this form 23.8 -> 23.3 ms, ResNet50 of 300 27.2 -> 27.1;
// with the GEMMs' too, ViT-S float32 step of 61 tiles 18.5 -> 17.6 ms, bf16 step of 37 tiles 3.71 -> 3.68.
#pragma once
#include "slide_internal.h"

namespace sl {

constexpr long long DMA_MAX = 0x70000000;   // no buffer is longer than this ...
constexpr int DMA_ABSENT = 0x78000000;      // ... so an element at this offset is outside of every one (with room for a small sum)

constexpr long long DMA_LD = 1 << 21;       // row stride up to which 128 rows of 4-byte elements fit one

// `bytes` (may be negative: nothing) from p on; both uniform
__device__ __forceinline__ __amdgpu_buffer_rsrc_t dma_buffer(const void* p, long long bytes) {
  const long long n = bytes > DMA_MAX ? DMA_MAX : bytes < 0 ? 0 : bytes;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)n, 0x00027000);
}
// `rows` rows of a matrix, at most 128: what lies behind the last one's `cols` columns is outside
template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t dma_rows(const T* p, int rows, int ld, int cols) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p), 0, rows > 0 ? ((rows - 1) * ld + cols) * (int)sizeof(T) : 0, 0x00027000);
}
// 16 bytes per lane from byte voff (per lane) + soff (uniform) of the buffer to 1 KB of consecutive LDS, lane l's at 16 l
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t b, void* lds, int voff, int soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(b, (__attribute__((address_space(3))) void*)lds, 16, voff, soff, 0, 0);
}

}  // namespace sl
