// Element-wise, layout and reduction kernels of the slide step (gfx950).
#include "slide_internal.h"

namespace sl {

// ---------------------------------------------------------------------------------------
// fp32 master weights [R,C] -> T copies [R,C] (bf16 path) and T transposes [C,R], every matrix of the encoder in one
// launch: a launch per matrix is 49 launches of 2 to 5 us for a 12-block encoder, more than the bytes take.
// ---------------------------------------------------------------------------------------
// workgroup -> matrix i of layer l, tile b of it; matrices 1 .. 4 repeat per layer
__device__ __forceinline__ void cast_tile(const CastTable& t, int& b, int& i, long long& l) {
  b = blockIdx.x; i = 0; l = 0;
  if (b >= t.blocks0) {
    b -= t.blocks0;
    l = b / t.blocks_layer;
    b -= (int)l * t.blocks_layer;
    i = 1;
    while (i < 4 && b >= t.m[i].blocks) { b -= t.m[i].blocks; ++i; }
  }
}

template <typename T>
__global__ void __launch_bounds__(256) cast_transpose_k(CastTable t, const float* __restrict__ params, char* __restrict__ shadow) {
  __shared__ float tile[32][33];
  int b, i;
  long long l;
  cast_tile(t, b, i, l);
  const CastTable::Mat m = t.m[i];
  const float* src = params + m.poff + l * t.stride_p;
  T* dstW = sizeof(T) == 4 ? nullptr : (T*)(shadow + m.w + l * t.stride_s);
  T* dstWT = (T*)(shadow + m.wt + l * t.stride_s);
  const int tc = (m.C + 31) / 32, c0 = b % tc * 32, r0 = b / tc * 32;
  int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
#pragma unroll
  for (int i = ty; i < 32; i += 8) {
    int r = r0 + i, c = c0 + tx;
    float v = (r < m.R && c < m.C) ? src[(size_t)r * m.C + c] : 0.f;
    tile[i][tx] = v;
    if (sizeof(T) == 2 && r < m.R && c < m.C) dstW[(size_t)r * m.C + c] = from_f<T>(v);
  }
  __syncthreads();
#pragma unroll
  for (int i = ty; i < 32; i += 8) {
    int c = c0 + i, r = r0 + tx;
    if (r < m.R && c < m.C) dstWT[(size_t)c * m.R + r] = from_f<T>(tile[tx][i]);
  }
}

// The bf16 copies by 64 x 64 tiles, every access along a row of 128 bytes (rows of a multiple of 8 elements, 16-byte addresses): bound by
// HBM.  TR: the transposes too, which only a backward reads.
// us (32 x 32 tiles, two bytes a lane, always with the transposes / this way): ViT-B 192 / 121 (5.6 TB/s), without transposes 90; ViT-S 52 / 34.
template <bool TR>
__global__ void __launch_bounds__(256) cast_tiles_k(CastTable t, const float* __restrict__ params, char* __restrict__ shadow) {
  constexpr int LD = 66;   // elements: an odd number of words
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  __shared__ __attribute__((aligned(16))) bf16 tile[64 * LD];
  int b, i;
  long long l;
  cast_tile(t, b, i, l);
  const CastTable::Mat m = t.m[i];
  const float* src = params + m.poff + l * t.stride_p;
  const int tc = (m.C + 63) / 64, c0 = b % tc * 64, r0 = b / tc * 64;
  bf16* W = (bf16*)(shadow + m.w + l * t.stride_s);
  const int lr = threadIdx.x >> 4, lc = (threadIdx.x & 15) * 4;
  float4 v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int r = r0 + lr + 16 * k, c = c0 + lc;
    v[k] = r < m.R && c < m.C ? *reinterpret_cast<const float4*>(src + (size_t)r * m.C + c) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int r = r0 + lr + 16 * k, c = c0 + lc;
    const bf16x4 h = {(bf16)v[k].x, (bf16)v[k].y, (bf16)v[k].z, (bf16)v[k].w};
    const u32x2 u = __builtin_bit_cast(u32x2, h);
    if (r < m.R && c < m.C) *reinterpret_cast<u32x2*>(W + (size_t)r * m.C + c) = u;
    if constexpr (TR) {
      unsigned* q = reinterpret_cast<unsigned*>(tile + (lr + 16 * k) * LD + lc);
      q[0] = u[0];
      q[1] = u[1];
    }
  }
  if constexpr (TR) {
    bf16* WT = (bf16*)(shadow + m.wt + l * t.stride_s);
    __syncthreads();
    const int rr = (threadIdx.x & 7) * 8;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int cc = (threadIdx.x >> 3) + 32 * k;
      bf16x8 h;
#pragma unroll
      for (int j = 0; j < 8; ++j) h[j] = tile[(rr + j) * LD + cc];
      if (c0 + cc < m.C && r0 + rr < m.R) *reinterpret_cast<u32x4*>(WT + (size_t)(c0 + cc) * m.R + r0 + rr) = __builtin_bit_cast(u32x4, h);
    }
  }
}

hipError_t launch_cast_transpose(int dt, CastTable t, int layers, const float* params, char* shadow, bool transposes, hipStream_t s) {
  if (dt == DT_F32 && !transposes) return hipSuccess;
  bool vec = dt == DT_BF16 && ((uintptr_t)params & 15) == 0 && ((uintptr_t)shadow & 15) == 0 && t.stride_p % 4 == 0 && t.stride_s % 16 == 0;
  for (int i = 0; i < 5; ++i) vec = vec && t.m[i].R % 8 == 0 && t.m[i].C % 8 == 0 && t.m[i].poff % 4 == 0 && t.m[i].w % 16 == 0 && t.m[i].wt % 16 == 0;
  const int side = vec ? 64 : 32;
  t.blocks_layer = 0;
  for (int i = 0; i < 5; ++i) {
    t.m[i].blocks = ((t.m[i].C + side - 1) / side) * ((t.m[i].R + side - 1) / side);
    if (i) t.blocks_layer += t.m[i].blocks;
  }
  t.blocks0 = t.m[0].blocks;
  const dim3 grid((unsigned)(t.blocks0 + (long long)layers * t.blocks_layer));
  if (vec) {
    if (transposes) hipLaunchKernelGGL(cast_tiles_k<true>, grid, dim3(256), 0, s, t, params, shadow);
    else hipLaunchKernelGGL(cast_tiles_k<false>, grid, dim3(256), 0, s, t, params, shadow);
  } else if (dt == DT_F32) hipLaunchKernelGGL(cast_transpose_k<float>, grid, dim3(256), 0, s, t, params, shadow);
  else hipLaunchKernelGGL(cast_transpose_k<bf16>, grid, dim3(256), 0, s, t, params, shadow);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// pixels [n,3,S,S] <-> patches [n*g*g, 3*P*P]   (patch order (gy,gx), flatten order (c,py,px))
// ---------------------------------------------------------------------------------------
// Patch matrix: tile n owns rows n * (g * g + lead) .. of 3 P P columns: `lead` rows of zeros (the slots of the tokens
// that are no patches, so that the matrix lines up row by row with the token matrix), then its g * g patches.
template <typename T>
__global__ void __launch_bounds__(256) patchify_k(const T* __restrict__ pix, T* __restrict__ pat, long long total,
                                                  int S, int P, int lead) {
  long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  int g = S / P, Kp = 3 * P * P;
  int col = (int)(i % Kp);
  long long row = i / Kp;
  int px = col % P, py = (col / P) % P, c = col / (P * P);
  int gx = (int)(row % g), gy = (int)((row / g) % g);
  long long n = row / (g * g);
  long long base = n * (g * g + lead);
  pat[(base + lead + row % (g * g)) * Kp + col] = pix[((n * 3 + c) * S + gy * P + py) * S + gx * P + px];
  if (row % (g * g) == 0)
    for (int l = 0; l < lead; ++l) pat[(base + l) * Kp + col] = from_f<T>(0.f);
}

// bf16, P % 8 == 0, S % 8 == 0: one workgroup per band of patches (tile n, patch row gy).  The band's 3 x P image
// rows are read with 16-byte accesses along the rows into LDS and written as whole patch rows, again 16 bytes
// per lane and contiguous (the element-wise kernel above moves 2 bytes per lane).
__global__ void __launch_bounds__(256) patchify_band_k(const bf16* __restrict__ pix, bf16* __restrict__ pat, int S, int P,
                                                       int lead) {
  extern __shared__ uint4 band[];   // [3 * P][S / 8] chunks of 8 pixels
  const int g = S / P, SC = S / 8, PC = P / 8, rows = 3 * P;
  const long long n = blockIdx.x / g;
  const int gy = blockIdx.x % g;
  for (int i = threadIdx.x; i < rows * SC; i += 256) {
    int r = i / SC, xc = i % SC, c = r / P, py = r % P;
    band[i] = *reinterpret_cast<const uint4*>(pix + ((n * 3 + c) * S + gy * P + py) * (long long)S + xc * 8);
  }
  __syncthreads();
  const int KC = rows * PC;          // chunks per patch row of the output
  bf16* out = pat + ((n * (g * g + lead) + lead) + gy * g) * (long long)(3 * P * P);
  if (gy == 0)   // the tile's leading rows of zeros
    for (int i = threadIdx.x; i < lead * KC; i += 256)
      *reinterpret_cast<uint4*>(pat + n * (g * g + lead) * (long long)(3 * P * P) + (long long)i * 8) = make_uint4(0, 0, 0, 0);
  for (int i = threadIdx.x; i < g * KC; i += 256) {
    int gx = i / KC, k = i % KC, r = k / PC, pc = k % PC;   // r = c * P + py
    *reinterpret_cast<uint4*>(out + (long long)i * 8) = band[r * SC + gx * PC + pc];
  }
}

template <typename T>
__global__ void __launch_bounds__(256) unpatchify_k(const T* __restrict__ dpat, T* __restrict__ dpix, long long total,
                                                    int S, int P, int lead) {
  long long i = (long long)blockIdx.x * 256 + threadIdx.x;  // index into dpix
  if (i >= total) return;
  int g = S / P, Kp = 3 * P * P;
  int x = (int)(i % S), y = (int)((i / S) % S), c = (int)((i / ((long long)S * S)) % 3);
  long long n = i / (3LL * S * S);
  long long row = n * (g * g + lead) + lead + (y / P) * g + x / P;
  int col = c * P * P + (y % P) * P + (x % P);
  dpix[i] = dpat[row * Kp + col];
}

// patchify_band_k the other way round: a band's patch rows into LDS with contiguous 16-byte reads, out as image rows
// (moving 2 bytes per lane, the kernel above ran at a third of the rate)
__global__ void __launch_bounds__(256) unpatchify_band_k(const bf16* __restrict__ dpat, bf16* __restrict__ dpix, int S, int P,
                                                         int lead) {
  extern __shared__ uint4 band[];   // [3 * P][S / 8] chunks of 8 pixels
  const int g = S / P, SC = S / 8, PC = P / 8, rows = 3 * P, KC = rows * PC;
  const long long n = blockIdx.x / g;
  const int gy = blockIdx.x % g;
  const bf16* in = dpat + ((n * (g * g + lead) + lead) + gy * g) * (long long)(3 * P * P);
  for (int i = threadIdx.x; i < g * KC; i += 256) {
    int gx = i / KC, k = i % KC, r = k / PC, pc = k % PC;   // r = c * P + py
    band[r * SC + gx * PC + pc] = *reinterpret_cast<const uint4*>(in + (long long)i * 8);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < rows * SC; i += 256) {
    int r = i / SC, xc = i % SC, c = r / P, py = r % P;
    *reinterpret_cast<uint4*>(dpix + ((n * 3 + c) * S + gy * P + py) * (long long)S + xc * 8) = band[i];
  }
}

static bool bands_ok(long long n, int S, int P) {   // P % 8 == 0, a whole number of patches, a band that fits 64 KB
  return P % 8 == 0 && S % P == 0 && n * (S / P) < (1LL << 31) && (size_t)3 * P * S * 2 <= 65536;
}

hipError_t launch_patchify(int dt, const void* pixels, void* patches, long long n, int S, int P, hipStream_t s, int lead) {
  long long total = n * 3LL * S * S;
  unsigned grid = (unsigned)((total + 255) / 256);
  if (dt == DT_F32)
    hipLaunchKernelGGL(patchify_k<float>, dim3(grid), dim3(256), 0, s, (const float*)pixels, (float*)patches, total, S, P, lead);
  else if (bands_ok(n, S, P))
    hipLaunchKernelGGL(patchify_band_k, dim3((unsigned)(n * (S / P))), dim3(256), (size_t)3 * P * S * 2, s,
                       (const bf16*)pixels, (bf16*)patches, S, P, lead);
  else
    hipLaunchKernelGGL(patchify_k<bf16>, dim3(grid), dim3(256), 0, s, (const bf16*)pixels, (bf16*)patches, total, S, P, lead);
  return hipGetLastError();
}

hipError_t launch_unpatchify(int dt, const void* dpatches, void* dpix, long long n, int S, int P, hipStream_t s, int lead) {
  long long total = n * 3LL * S * S;
  unsigned grid = (unsigned)((total + 255) / 256);
  if (dt == DT_F32)
    hipLaunchKernelGGL(unpatchify_k<float>, dim3(grid), dim3(256), 0, s, (const float*)dpatches, (float*)dpix, total, S, P, lead);
  else if (bands_ok(n, S, P) && ((uintptr_t)dpix & 15) == 0)
    hipLaunchKernelGGL(unpatchify_band_k, dim3((unsigned)(n * (S / P))), dim3(256), (size_t)3 * P * S * 2, s,
                       (const bf16*)dpatches, (bf16*)dpix, S, P, lead);
  else
    hipLaunchKernelGGL(unpatchify_k<bf16>, dim3(grid), dim3(256), 0, s, (const bf16*)dpatches, (bf16*)dpix, total, S, P, lead);
  return hipGetLastError();
}

// x[n, 0, :] = cls + pos[0]
template <typename RS>
__global__ void __launch_bounds__(256) cls_rows_k(RS* __restrict__ x, const float* __restrict__ cls,
                                                  const float* __restrict__ pos, long long n, int T, int D) {
  long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n * D) return;
  int d = (int)(i % D);
  long long t = i / D;
  x[t * T * D + d] = from_f<RS>(cls[d] + pos[d]);
}

hipError_t launch_cls_rows(int dt, void* x, const float* cls, const float* pos, long long n, int T, int D, hipStream_t s) {
  unsigned grid = (unsigned)((n * D + 255) / 256);
  if (dt == DT_F32)
    hipLaunchKernelGGL(cls_rows_k<float>, dim3(grid), dim3(256), 0, s, (float*)x, cls, pos, n, T, D);
  else
    hipLaunchKernelGGL(cls_rows_k<rs_bf16path_t>, dim3(grid), dim3(256), 0, s, (rs_bf16path_t*)x, cls, pos, n, T, D);
  return hipGetLastError();
}

// The rows the patch embedding adds to its product, one per token position, as the residual-stream type:
// tab[0] = cls + pos[0] (the patch matrix has a row of zeros there), tab[t] = bias + pos[t] for the patch tokens.
__global__ void __launch_bounds__(256) pos_table_k(rs_bf16path_t* __restrict__ tab, const float* __restrict__ cls,
                                                   const float* __restrict__ pos, const float* __restrict__ bias, int T, int D) {
  int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= T * D) return;
  int d = i % D;
  tab[i] = from_f<rs_bf16path_t>(pos[i] + (i < D ? cls[d] : bias[d]));
}

hipError_t launch_pos_table(void* tab, const float* cls, const float* pos, const float* bias, int T, int D, hipStream_t s) {
  hipLaunchKernelGGL(pos_table_k, dim3((unsigned)((T * D + 255) / 256)), dim3(256), 0, s, (rs_bf16path_t*)tab, cls, pos, bias, T, D);
  return hipGetLastError();
}

// zero fill in 16-byte words (bytes must be a multiple of 16; all arena regions are)
__global__ void __launch_bounds__(256) fill_zero_k(uint4* __restrict__ p, size_t words) {
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  size_t stride = (size_t)gridDim.x * 256;
  for (; i < words; i += stride) p[i] = make_uint4(0, 0, 0, 0);
}

// plain copy, 16 bytes per lane, grid-stride: the known-size kernel that hardware traffic counters are scaled with
__global__ void __launch_bounds__(256) calib_copy_k(uint4* __restrict__ dst, const uint4* __restrict__ src, size_t words) {
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x, step = (size_t)gridDim.x * 256;
  for (; i < words; i += step) dst[i] = src[i];
}

hipError_t launch_calib_copy(void* dst, const void* src, size_t bytes, hipStream_t s) {
  size_t words = bytes / 16;
  if (!words) return hipSuccess;
  size_t blocks = (words + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(calib_copy_k, dim3((unsigned)blocks), dim3(256), 0, s, (uint4*)dst, (const uint4*)src, words);
  return hipGetLastError();
}

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s) {
  size_t words = bytes / 16;
  if (words == 0) return hipSuccess;
  size_t blocks = (words + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(fill_zero_k, dim3((unsigned)blocks), dim3(256), 0, s, (uint4*)p, words);
  return hipGetLastError();
}

template <typename T>
__global__ void __launch_bounds__(256) gelu_k(const T* __restrict__ m, T* __restrict__ a, long long count) {
  long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  long long stride = (long long)gridDim.x * 256;
  for (; i < count; i += stride) a[i] = from_f<T>(gelu_f(to_f(m[i])));
}

hipError_t launch_gelu(int dt, const void* m, void* a, long long count, hipStream_t s) {
  long long blocks = (count + 255) / 256;
  if (blocks > 262144) blocks = 262144;
  if (blocks == 0) return hipSuccess;
  if (dt == DT_F32)
    hipLaunchKernelGGL(gelu_k<float>, dim3((unsigned)blocks), dim3(256), 0, s, (const float*)m, (float*)a, count);
  else
    hipLaunchKernelGGL(gelu_k<bf16>, dim3((unsigned)blocks), dim3(256), 0, s, (const bf16*)m, (bf16*)a, count);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// column sums, two-stage and deterministic: part[s][c] = sum over rows of slab s
// ---------------------------------------------------------------------------------------
template <typename E>
__global__ void __launch_bounds__(256) colsum_k(const E* __restrict__ A, long long lda, RowMap map, long long M, int N,
                                                float* __restrict__ part, int slabs) {
  __shared__ float red[4][64];
  int cl = threadIdx.x & 63, q = threadIdx.x >> 6;
  int c = blockIdx.x * 64 + cl;
  int s = blockIdx.y;
  long long per = (M + slabs - 1) / slabs;
  long long lo = (long long)s * per, hi = lo + per < M ? lo + per : M;
  float acc = 0.f;
  if (c < N)
    for (long long r = lo + q; r < hi; r += 4) acc += to_f(A[map(r) * lda + c]);
  red[q][cl] = acc;
  __syncthreads();
  if (q == 0 && c < N) part[(size_t)s * N + c] = (red[0][cl] + red[1][cl]) + (red[2][cl] + red[3][cl]);
}

// The same sums for bf16 rows read 16 bytes per lane (a lane owns 8 neighbouring columns), four rows of a quarter in
// flight: the element-wise kernel above moves 2 bytes per lane and load, which is a third of the memory rate on the
// position gradient (a [tiles] x [T * D] matrix, 1.2 GB on the 8192-tile slide).  Identity row map, N and lda
// multiples of 8, 16-byte aligned rows.  Fixed order of additions (four chains per element, combined pairwise).
__global__ void __launch_bounds__(256) colsum8_k(const bf16* __restrict__ A, long long lda, long long M, int N,
                                                 float* __restrict__ part, int slabs) {
  __shared__ float red[4][64][9];
  typedef unsigned int cu4 __attribute__((ext_vector_type(4)));
  const int cl = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int c = (blockIdx.x * 64 + cl) * 8;
  const int s = blockIdx.y;
  const long long per = (M + slabs - 1) / slabs;
  const long long lo = (long long)s * per, hi = lo + per < M ? lo + per : M;
  float acc[4][8];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[u][e] = 0.f;
  if (c < N) {
    long long r = lo + q;
    for (; r + 12 < hi; r += 16) {
      cu4 t[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) t[u] = __builtin_nontemporal_load(reinterpret_cast<const cu4*>(A + (r + 4 * u) * lda + c));
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          acc[u][2 * w] += __uint_as_float(t[u][w] << 16);
          acc[u][2 * w + 1] += __uint_as_float(t[u][w] & 0xffff0000u);
        }
    }
    for (; r < hi; r += 4) {
      cu4 t = *reinterpret_cast<const cu4*>(A + r * lda + c);
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        acc[0][2 * w] += __uint_as_float(t[w] << 16);
        acc[0][2 * w + 1] += __uint_as_float(t[w] & 0xffff0000u);
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) red[q][cl][e] = (acc[0][e] + acc[1][e]) + (acc[2][e] + acc[3][e]);
  __syncthreads();
  if (q == 0 && c < N) {
#pragma unroll
    for (int e = 0; e < 8; ++e) part[(size_t)s * N + c + e] = (red[0][cl][e] + red[1][cl][e]) + (red[2][cl][e] + red[3][cl][e]);
  }
}

int colsum_slabs(long long M) {
  long long s = (M + 511) / 512;
  if (s < 1) s = 1;
  if (s > 128) s = 128;
  return (int)s;
}

// Sums over slab partials, any number of results in one launch (a launch per weight, bias, gain and shift gradient is nine
// per block of the encoder, most of them shorter than a launch).  The additions of a result have a fixed order that does not
// depend on scheduling.  A result's kind says how its outputs and slabs are dealt to a workgroup:
//   RED_F   1024 outputs, four neighbours per thread, which adds the slabs itself: long results of up to 8 slabs, which are all in
//           flight together.  As RED_4 five blocks' weights of ViT-S are 35,262 workgroups, 94 us at 5 slabs (9,342 and 48 this way);
//           with 16 slabs (fc1 and fc2 of 16 tiles in float32) a RED_4 workgroup has work enough, and the two measured the same
//   RED_4   256 outputs, four neighbours per thread (16-byte accesses), slabs dealt to 4 quarter groups, in the same order
//   RED_1   64 outputs, otherwise the same
//   RED_16  16 outputs, slabs dealt to 16 groups of lanes (short results of up to a thousand slabs), the 16 group sums added
//           as a binary tree
__global__ void __launch_bounds__(256) reduce_partials_k(RedList L) {
  __shared__ float4 red4[4][64];
  int i = 0;
  while (i + 1 < L.n && (int)blockIdx.x >= L.seg[i + 1].block0) ++i;
  const RedSeg sg = L.seg[i];
  const float* __restrict__ part = sg.part;
  const long long b = blockIdx.x - sg.block0;
  if (sg.kind == RED_F) {
    const long long o = (b * 256 + threadIdx.x) * 4;
    if (o >= sg.len) return;
    const f32x4* p = reinterpret_cast<const f32x4*>(part + o);
    const long long st = sg.stride >> 2;
    const f32x4 t = sg.accumulate ? *reinterpret_cast<const f32x4*>(sg.out + o) : f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 a[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < sg.slabs; s0 += 8) {   // uniform; once (without the loop the compiler takes 202 registers)
      f32x4 v[8];
#pragma unroll
      for (int s = 0; s < 8; ++s)
        if (s0 + s < sg.slabs) v[s] = p[(s0 + s) * st];
#pragma unroll
      for (int s = 0; s < 8; ++s)
        if (s0 + s < sg.slabs) a[s & 3] += v[s];
    }
    f32x4 r = (a[0] + a[1]) + (a[2] + a[3]);
    if (sg.accumulate) r += t;
    *reinterpret_cast<f32x4*>(sg.out + o) = r;
  } else if (sg.kind == RED_4) {
    const int cl = threadIdx.x & 63, q = threadIdx.x >> 6;
    const long long o = (b * 64 + cl) * 4;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    if (o < sg.len) {
#pragma unroll 4
      for (int s = q; s < sg.slabs; s += 4) {
        float4 v = *reinterpret_cast<const float4*>(part + (size_t)s * sg.stride + o);
        acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
      }
    }
    red4[q][cl] = acc;
    __syncthreads();
    if (q == 0 && o < sg.len) {
      float4 x = red4[0][cl], y = red4[1][cl], z = red4[2][cl], w = red4[3][cl];
      float4 v = make_float4((x.x + y.x) + (z.x + w.x), (x.y + y.y) + (z.y + w.y), (x.z + y.z) + (z.z + w.z),
                             (x.w + y.w) + (z.w + w.w));
      float4* out = reinterpret_cast<float4*>(sg.out + o);
      if (sg.accumulate) { float4 t = *out; v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w; }
      *out = v;
    }
  } else if (sg.kind == RED_1) {
    float (*red)[64] = reinterpret_cast<float (*)[64]>(red4);
    const int cl = threadIdx.x & 63, q = threadIdx.x >> 6;
    const long long o = b * 64 + cl;
    float acc = 0.f;
    if (o < sg.len) {
#pragma unroll 4
      for (int s = q; s < sg.slabs; s += 4) acc += part[(size_t)s * sg.stride + o];
    }
    red[q][cl] = acc;
    __syncthreads();
    if (q == 0 && o < sg.len) {
      float v = (red[0][cl] + red[1][cl]) + (red[2][cl] + red[3][cl]);
      sg.out[o] = sg.accumulate ? sg.out[o] + v : v;
    }
  } else {
    float (*red)[17] = reinterpret_cast<float (*)[17]>(red4);
    const int cl = threadIdx.x & 15, q = threadIdx.x >> 4;
    const long long o = b * 16 + cl;
    float a0 = 0.f, a1 = 0.f;
    if (o < sg.len) {
      int s = q;
#pragma unroll 4
      for (; s + 16 < sg.slabs; s += 32) {
        a0 += part[(size_t)s * sg.stride + o];
        a1 += part[(size_t)(s + 16) * sg.stride + o];
      }
      if (s < sg.slabs) a0 += part[(size_t)s * sg.stride + o];
    }
    red[q][cl] = a0 + a1;
    __syncthreads();
    if (q == 0 && o < sg.len) {
      float t[16];
#pragma unroll
      for (int g = 0; g < 16; ++g) t[g] = red[g][cl];
#pragma unroll
      for (int w = 8; w > 0; w >>= 1)
#pragma unroll
        for (int g = 0; g < w; ++g) t[g] += t[g + w];
      sg.out[o] = sg.accumulate ? sg.out[o] + t[0] : t[0];
    }
  }
}

bool red_add(RedList& L, const float* part, int slabs, long long stride, long long len, float* out, int accumulate) {
  if (len <= 0) return true;
  if (L.n >= RED_MAX) return false;
  RedSeg& g = L.seg[L.n];
  g.part = part; g.out = out; g.stride = stride; g.len = (int)len; g.slabs = slabs; g.accumulate = accumulate != 0;
  if (len < 4096 && slabs >= 64) g.kind = RED_16;
  else if (len >= 4096 && len % 4 == 0 && stride % 4 == 0 && ((uintptr_t)part & 15) == 0 && ((uintptr_t)out & 15) == 0)
    g.kind = slabs <= 8 && len >= 65536 ? RED_F : RED_4;
  else g.kind = RED_1;
  g.block0 = L.blocks;
  const int per = g.kind == RED_16 ? 16 : g.kind == RED_F ? 1024 : g.kind == RED_4 ? 256 : 64;
  L.blocks += (int)((len + per - 1) / per);
  ++L.n;
  return true;
}

hipError_t launch_reduce_partials(const RedList& L, hipStream_t s) {
  if (L.n == 0) return hipSuccess;
  hipLaunchKernelGGL(reduce_partials_k, dim3((unsigned)L.blocks), dim3(256), 0, s, L);
  return hipGetLastError();
}

hipError_t launch_colsum_part(int elem, const void* A, long long lda, RowMap map, long long M, int N, float* part,
                              int slabs, hipStream_t s) {
  if (elem != DT_F32 && map.g2 == 0 && N % 8 == 0 && lda % 8 == 0 && ((size_t)A & 15) == 0 && M >= 64) {
    hipLaunchKernelGGL(colsum8_k, dim3((N / 8 + 63) / 64, slabs), dim3(256), 0, s, (const bf16*)A, lda, M, N, part, slabs);
    return hipGetLastError();
  }
  dim3 grid((N + 63) / 64, slabs);
  if (elem == DT_F32)
    hipLaunchKernelGGL(colsum_k<float>, grid, dim3(256), 0, s, (const float*)A, lda, map, M, N, part, slabs);
  else
    hipLaunchKernelGGL(colsum_k<bf16>, grid, dim3(256), 0, s, (const bf16*)A, lda, map, M, N, part, slabs);
  return hipGetLastError();
}

}  // namespace sl
