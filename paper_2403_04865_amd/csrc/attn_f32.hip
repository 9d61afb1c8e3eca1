// Softmax attention inside one tile in float32 on the matrix cores (v_mfma_f32_32x32x2_f32), head dimension 32 or 64.
//
// A workgroup belongs to one (tile, head) and keeps the two operands that its wavefronts sweep over in LDS (keys and
// values forward and for dQ; queries and dO for dK and dV), rows padded by four floats so that 16-byte reads of 16
// consecutive rows fall on 64 different banks.  A wavefront owns a block of 32 queries (or keys) as the columns of its
// products: the scores come out with that block's index in the lane, which is exactly how the next product wants them as
// an operand, so probabilities and their gradients never leave the registers:
//   forward   S^T = K Q^T,  online softmax down the columns,  O^T += V^T P^T
//   dQ        S^T = K Q^T,  dP^T = V dO^T,  dS^T = P^T (dP^T - delta),  dQ^T += K^T dS^T
//   dK, dV    S = Q K^T,  dP = dO V^T,  dV^T += dO^T P,  dK^T += Q^T dS
// The matrix pipe bounds it (256 flops a clock and compute unit in float32); one or two wavefronts per SIMD are what the
// 100 KB of operands of 197 tokens leave room for.
#include "slide_internal.h"

namespace sl {

namespace {

constexpr int PAD = 4;

__device__ __forceinline__ f32x16 mfma(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}
__device__ __forceinline__ f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

// rows 0 .. Tn - 1 of a [.., ld] matrix into [TP][DH + PAD], zeros behind them
template <int DH>
__device__ __forceinline__ void stage(float* dst, const float* src, long long ld, int Tn, int TP, float scale) {
  constexpr int V = DH / 4;
  for (int i = threadIdx.x; i < TP * V; i += blockDim.x) {
    const int j = i / V, e = (i % V) * 4;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (j < Tn) v = ld4(src + j * ld + e) * scale;
    *reinterpret_cast<f32x4*>(dst + j * (DH + PAD) + e) = v;
  }
}

// this lane's half of a row as an MFMA operand: floats 8 s + 4 (lane / 32) .. + 3 for s = 0 .. DH / 8 - 1
template <int DH>
__device__ __forceinline__ void frag(f32x4 (&f)[DH / 8], const float* row, bool ok, int half, float scale) {
#pragma unroll
  for (int s = 0; s < DH / 8; ++s) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (ok) v = ld4(row + 8 * s + 4 * half) * scale;
    f[s] = v;
  }
}

// 32 x 32 block: rows = rows `row0 + lane % 32` of X (LDS), columns = the block whose operand is f
template <int DH>
__device__ __forceinline__ f32x16 scores(const float* X, const f32x4 (&f)[DH / 8], int row, int half) {
  f32x16 acc = zero16();
  const float* x = X + row * (DH + PAD) + 4 * half;
#pragma unroll
  for (int s = 0; s < DH / 8; ++s) {
    const f32x4 a = ld4(x + 8 * s);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = mfma(a[e], f[s][e], acc);
  }
  return acc;
}

// acc[nb]^T += X[row0 ..]^T p: rows of the result are columns nb * 32 .. of X; element r of p belongs to row (r / 4) * 8 + 4 half + r % 4
template <int DH>
__device__ __forceinline__ void accumulate(f32x16 (&acc)[DH / 32], const float* X, const f32x16& p, int row0, int col, int half) {
  const float* x = X + (row0 + 4 * half) * (DH + PAD) + col;
#pragma unroll
  for (int r = 0; r < 16; ++r)
#pragma unroll
    for (int nb = 0; nb < DH / 32; ++nb) acc[nb] = mfma(x[((r >> 2) * 8 + (r & 3)) * (DH + PAD) + nb * 32], p[r], acc[nb]);
}

template <int DH>
__device__ __forceinline__ void store_t(float* row, const f32x16 (&acc)[DH / 32], int half, float scale) {
#pragma unroll
  for (int nb = 0; nb < DH / 32; ++nb)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4 v = {acc[nb][4 * q], acc[nb][4 * q + 1], acc[nb][4 * q + 2], acc[nb][4 * q + 3]};
      *reinterpret_cast<f32x4*>(row + nb * 32 + q * 8 + half * 4) = v * scale;
    }
}

// grid (tiles * H, parts): part y takes the query blocks y * W + w, W wavefronts; cls_only: query block 0 only
template <int DH>
__global__ void __launch_bounds__(512) attn_fwd_f32_k(const float* __restrict__ qkv, float* __restrict__ O, float* __restrict__ lse,
                                                      int Tn, int H, int cls_only) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int TP = (Tn + 31) & ~31, h = blockIdx.x % H;
  const long long tile = blockIdx.x / H;
  const int D = H * DH;
  const float* base = qkv + tile * Tn * 3LL * D + h * DH;
  float *Ks = lds, *Vs = lds + TP * (DH + PAD);
  stage<DH>(Ks, base + D, 3LL * D, Tn, TP, 1.f);
  stage<DH>(Vs, base + 2 * D, 3LL * D, Tn, TP, 1.f);
  const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
  const int qb = blockIdx.y * (blockDim.x >> 6) + (threadIdx.x >> 6), i = qb * 32 + col;
  f32x4 qf[DH / 8];
  frag<DH>(qf, base + (long long)i * 3 * D, i < Tn, half, 1.0f / sqrtf((float)DH));
  __syncthreads();
  if (qb * 32 >= Tn || (cls_only && qb > 0)) return;
  f32x16 o[DH / 32];
#pragma unroll
  for (int nb = 0; nb < DH / 32; ++nb) o[nb] = zero16();
  float m = -INFINITY, l = 0.f;
  for (int k0 = 0; k0 < TP; k0 += 32) {
    f32x16 s = scores<DH>(Ks, qf, k0 + col, half);
    if (k0 + 32 > Tn) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (k0 + (r >> 2) * 8 + half * 4 + (r & 3) >= Tn) s[r] = -INFINITY;
    }
    float bm = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) bm = fmaxf(bm, s[r]);
    bm = fmaxf(bm, __shfl_xor(bm, 32, 64));
    const float mn = fmaxf(m, bm), al = __expf(m - mn);   // every block has at least one key: mn is finite
    m = mn;
    l *= al;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = __expf(s[r] - mn);
      l += s[r];
    }
#pragma unroll
    for (int nb = 0; nb < DH / 32; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[nb][r] *= al;
    accumulate<DH>(o, Vs, s, k0, col, half);
  }
  l += __shfl_xor(l, 32, 64);
  if (i >= Tn) return;
  store_t<DH>(O + (tile * Tn + i) * D + h * DH, o, half, 1.0f / l);
  if (half == 0) lse[(tile * H + h) * Tn + i] = m + logf(l);
}

// grid (tiles * H, 2 * parts): even y the dQ of a part's query blocks, odd y the dK and dV of its key blocks.  cls_only: query 0
// alone carries an output gradient (no other row of dO is read), dQ is zero for every other query
template <int DH>
__global__ void __launch_bounds__(512) attn_bwd_f32_k(const float* __restrict__ qkv, const float* __restrict__ O,
                                                      const float* __restrict__ lse, const float* __restrict__ dO,
                                                      float* __restrict__ dqkv, int Tn, int H, int cls_only) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int TP = (Tn + 31) & ~31, h = blockIdx.x % H;
  const long long tile = blockIdx.x / H;
  const int D = H * DH;
  const float* base = qkv + tile * Tn * 3LL * D + h * DH;
  float* dbase = dqkv + tile * Tn * 3LL * D + h * DH;
  const float* ob = O + tile * Tn * (long long)D + h * DH;
  const float* gob = dO + tile * Tn * (long long)D + h * DH;
  const float* lb = lse + (tile * H + h) * Tn;
  const float scale = 1.0f / sqrtf((float)DH);
  float *Xs = lds, *Ys = lds + TP * (DH + PAD), *ls = Ys + TP * (DH + PAD), *dl = ls + TP;
  const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
  const int blk = (blockIdx.y >> 1) * (blockDim.x >> 6) + (threadIdx.x >> 6), i = blk * 32 + col;
  const bool ok = i < Tn, gok = cls_only ? i == 0 : ok;   // rows that exist, rows of dO that are defined
  const int TG = cls_only ? 1 : Tn, TQ = cls_only ? 32 : TP;
  if ((blockIdx.y & 1) == 0) {
    if (cls_only && blockIdx.y) {   // uniform: later blocks of queries
      if (ok) {
        const f32x16 z[DH / 32] = {};
        store_t<DH>(dbase + (long long)i * 3 * D, z, half, 1.f);
      }
      return;
    }
    stage<DH>(Xs, base + D, 3LL * D, Tn, TP, 1.f);
    stage<DH>(Ys, base + 2 * D, 3LL * D, Tn, TP, 1.f);
    f32x4 qf[DH / 8], gf[DH / 8];
    frag<DH>(qf, base + (long long)i * 3 * D, ok, half, scale);
    frag<DH>(gf, gob + (long long)i * D, gok, half, 1.f);
    float delta = 0.f;
#pragma unroll
    for (int s = 0; s < DH / 8; ++s)
      if (gok) {
        const f32x4 t = ld4(ob + (long long)i * D + 8 * s + 4 * half) * gf[s];
        delta += (t[0] + t[1]) + (t[2] + t[3]);
      }
    delta += __shfl_xor(delta, 32, 64);
    const float li = ok ? lb[i] : 0.f;
    __syncthreads();
    if (blk * 32 >= Tn) return;
    f32x16 dq[DH / 32];
#pragma unroll
    for (int nb = 0; nb < DH / 32; ++nb) dq[nb] = zero16();
    for (int k0 = 0; k0 < (cls_only && blk > 0 ? 0 : TP); k0 += 32) {
      f32x16 s = scores<DH>(Xs, qf, k0 + col, half);
      const f32x16 dp = scores<DH>(Ys, gf, k0 + col, half);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = k0 + (r >> 2) * 8 + half * 4 + (r & 3) < Tn ? __expf(s[r] - li) : 0.f;
        s[r] = p * (dp[r] - delta);
      }
      accumulate<DH>(dq, Xs, s, k0, col, half);
    }
    if (ok) store_t<DH>(dbase + (long long)i * 3 * D, dq, half, scale);
    return;
  }
  stage<DH>(Xs, base, 3LL * D, Tn < TQ ? Tn : TQ, TQ, scale);
  stage<DH>(Ys, gob, D, TG, TQ, 1.f);
  for (int j = threadIdx.x; j < TQ; j += blockDim.x) ls[j] = j < Tn ? lb[j] : INFINITY;   // queries past the end: P = 0
  constexpr int V = DH / 4;
  for (int k = threadIdx.x; k < TQ * V; k += blockDim.x) {   // V neighbouring lanes share a row, TQ * V is a multiple of 64
    const int j = k / V, e = (k % V) * 4;
    float d = 0.f;
    if (j < TG) {
      const f32x4 t = ld4(gob + (long long)j * D + e) * ld4(ob + (long long)j * D + e);
      d = (t[0] + t[1]) + (t[2] + t[3]);
    }
#pragma unroll
    for (int o = V / 2; o > 0; o >>= 1) d += __shfl_xor(d, o, 64);
    if (e == 0) dl[j] = d;
  }
  f32x4 kf[DH / 8], vf[DH / 8];
  frag<DH>(kf, base + D + (long long)i * 3 * D, ok, half, 1.f);
  frag<DH>(vf, base + 2 * D + (long long)i * 3 * D, ok, half, 1.f);
  __syncthreads();
  if (blk * 32 >= Tn) return;
  f32x16 dk[DH / 32], dv[DH / 32];
#pragma unroll
  for (int nb = 0; nb < DH / 32; ++nb) dk[nb] = dv[nb] = zero16();
  for (int q0 = 0; q0 < TQ; q0 += 32) {
    f32x16 p = scores<DH>(Xs, kf, q0 + col, half);
    f32x16 ds = scores<DH>(Ys, vf, q0 + col, half);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 l4 = ld4(ls + q0 + q * 8 + half * 4), d4 = ld4(dl + q0 + q * 8 + half * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = 4 * q + e;
        p[r] = __expf(p[r] - l4[e]);
        ds[r] = p[r] * (ds[r] - d4[e]);
      }
    }
    accumulate<DH>(dv, Ys, p, q0, col, half);
    accumulate<DH>(dk, Xs, ds, q0, col, half);   // Xs holds q * scale
  }
  if (ok) {
    store_t<DH>(dbase + D + (long long)i * 3 * D, dk, half, 1.f);
    store_t<DH>(dbase + 2 * D + (long long)i * 3 * D, dv, half, 1.f);
  }
}

size_t lds_bytes(int T, int dh) {
  const size_t TP = (size_t)((T + 31) & ~31);
  return (2 * TP * (dh + PAD) + 2 * TP) * sizeof(float);
}

template <typename K>
hipError_t set_lds(K kernel, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// Wavefronts per workgroup (one workgroup of 197 tokens fits a compute unit): four, a block of 32 each, while the workgroups
// that makes find a compute unit each, else up to eight, two per SIMD.  197 tokens, 6 heads, four / eight: 20 tiles forward
// 26 / 38 us, backward 97 / 74; 61 tiles 88 / 81 and 276 / 204 (vector kernels: 375 and 1145).
int waves(long long heads, int blocks, int roles) {
  const int w = blocks < 4 ? blocks : 4;
  if (heads * ((blocks + w - 1) / w) * roles <= 256) return w;
  return blocks < 8 ? blocks : 8;
}

}  // namespace

bool attn_f32_ok(int T, int dh) { return (dh == 64 || dh == 32) && lds_bytes(T, dh) <= 160 * 1024; }

hipError_t launch_attn_fwd_f32(const float* qkv, float* O, float* lse, long long n, int T, int H, int dh, int cls_only, hipStream_t s) {
  const int nb = (T + 31) / 32, w = cls_only ? (nb < 4 ? nb : 4) : waves(n * H, nb, 1);
  const size_t lds = lds_bytes(T, dh);
  if (n * H >= (1LL << 31)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(n * H), cls_only ? 1 : (nb + w - 1) / w), block(64 * w);
  hipError_t e = dh == 64 ? set_lds(attn_fwd_f32_k<64>, lds) : set_lds(attn_fwd_f32_k<32>, lds);
  if (e != hipSuccess) return e;
  if (dh == 64) hipLaunchKernelGGL(attn_fwd_f32_k<64>, grid, block, lds, s, qkv, O, lse, T, H, cls_only);
  else hipLaunchKernelGGL(attn_fwd_f32_k<32>, grid, block, lds, s, qkv, O, lse, T, H, cls_only);
  return hipGetLastError();
}

hipError_t launch_attn_bwd_f32(const float* qkv, const float* O, const float* lse, const float* dO, float* dqkv, long long n,
                               int T, int H, int dh, int cls_only, hipStream_t s) {
  const int nb = (T + 31) / 32, w = waves(n * H, nb, 2);
  const size_t lds = lds_bytes(T, dh);
  if (n * H >= (1LL << 31)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(n * H), 2 * ((nb + w - 1) / w)), block(64 * w);
  hipError_t e = dh == 64 ? set_lds(attn_bwd_f32_k<64>, lds) : set_lds(attn_bwd_f32_k<32>, lds);
  if (e != hipSuccess) return e;
  if (dh == 64) hipLaunchKernelGGL(attn_bwd_f32_k<64>, grid, block, lds, s, qkv, O, lse, dO, dqkv, T, H, cls_only);
  else hipLaunchKernelGGL(attn_bwd_f32_k<32>, grid, block, lds, s, qkv, O, lse, dO, dqkv, T, H, cls_only);
  return hipGetLastError();
}

}  // namespace sl
