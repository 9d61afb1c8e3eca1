// Gated-attention MIL pooling over the feature rows in float32 on the matrix cores: every shape and row count that has no
// bf16 kernel (float32 path, short bags, feature widths of the convolutional encoders, the backward at D = 768).
//
// The three contractions are taken as blocks of 32 rows x 32 gate units (or features), one per workgroup, with the
// contracted index dealt to the workgroup's wavefronts and their partial blocks added through LDS: a bag of 16 to 1,000
// rows is a few thousand MFMAs altogether and what bounds it is the serial chain of one wavefront, so the work is cut
// along all three indices.  (One workgroup per 16 rows with all gate units on the vector units, one dot product per
// wavefront at a time: 37 x 384 rows, M_h = 128 209 us forward and 279 us backward, now 11 and 20.)  Rows wider than 1536
// features have kernels of their own (below).
// MFMA operands come straight from global memory: a lane reads four consecutive elements of its row and gives one to each
// of four MFMAs (which index an MFMA contracts does not matter as long as both operands agree).  Weights are the first
// operand: a lane then owns one feature row and runs of four neighbouring gate units (features).
#include "slide_internal.h"
#include "split_f32.h"

namespace sl {

namespace {

constexpr int U = 6;   // steps of a contraction whose loads are issued together

__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}

// elements k .. k + 3 of a row of n, zeros behind its end; VEC: n and the row's address allow 16-byte reads
template <bool VEC>
__device__ __forceinline__ f32x4 ld4(const float* row, int k, int n) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if constexpr (VEC) {
    if (k < n) v = *reinterpret_cast<const f32x4*>(row + k);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (k + e < n) v[e] = row[k + e];
  }
  return v;
}

// Pre-activations of 32 rows x 32 gate units of V and of U, K split over the wavefronts, then per element
//   forward   w t s summed over a block's gate units: part[blockIdx.y][n], or over all of them, block by block in the order
//             in which the parts would be added, where there is room for one part only (gridDim.y = 1): the same bits
//   backward  Dp[n] = [dpV | dpU] (2 M_h), dwp[blockIdx.x][j] = sum over the 32 rows of da t s
// where t = tanh(V h + b_V), s = sigmoid(U h + b_U), da_n = alpha_n dz . (h_n - z).  All of it stays float32: the column
// sums of the backward's terms cancel almost completely (the da of a slide add up to zero).
template <bool VEC, bool BWD>
__global__ void __launch_bounds__(512) pool_gate_f32_k(PoolArgs p, float* __restrict__ out, float* __restrict__ dwp) {
  extern __shared__ float red[];   // [W][32][64] partial blocks, then [W][64] dot products / partial logits
  const int W = blockDim.x >> 6, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 31, half = lane >> 5;
  const int D = p.D, Mh = p.Mh, nc = (D + 7) / 8;
  // The backward takes its pre-activations and dot products in shorter chains of additions: what a row is off by stays in the
  // gate gradients, whose terms cancel.  Their error against 64 bits, geometric mean over 15 bags of 5 to 8,192 rows, is 0.81
  // (V.b) to 0.86 (w) of what it is with one chain per wavefront.  (The forward took 5 % longer with two at 100 rows.)
  constexpr int NA = BWD ? 2 : 1;
  float* aux = red + W * 32 * 64;
  const long long n = (long long)blockIdx.x * 32 + li;
  const bool ok = n < p.N;
  const float* hrow = p.H + (ok ? n : p.N - 1) * D;
  const float* zv = p.scal + pool_z_off(p.C);
  if (!BWD && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *p.ticket = 0;
  float logit = 0.f;   // threads 0 .. 31
  for (int ub = blockIdx.y; ub * 32 < Mh; ub += gridDim.y) {
    const int u = ub * 32 + li < Mh ? ub * 32 + li : Mh - 1;
    const float *vr = p.VW + (size_t)u * D, *ur = p.UW + (size_t)u * D;
    f32x16 av[NA], au[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) av[i] = au[i] = zero16();
    float dot = 0.f, part = 0.f;
    for (int c0 = wave; c0 < nc; c0 += U * W) {   // U steps' loads in flight
      f32x4 h[U], v[U], w[U];
#pragma unroll
      for (int i = 0; i < U; ++i) {
        const int k = (c0 + i * W) * 8 + half * 4;
        h[i] = ld4<VEC>(hrow, k, D);
        v[i] = ld4<VEC>(vr, k, D);
        w[i] = ld4<VEC>(ur, k, D);
      }
#pragma unroll
      for (int i = 0; i < U; ++i)
        if (c0 + i * W < nc) {
          if constexpr (BWD) {
            const int k = (c0 + i * W) * 8 + half * 4;
            const f32x4 z = ld4<VEC>(zv, k, D), dz = ld4<VEC>(zv + D, k, D), zl = ld4<VEC>(zv + 2 * D, k, D);
            const f32x4 t = ((h[i] - z) - zl) * dz;
            dot += (t[0] + t[1]) + (t[2] + t[3]);
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            av[e % NA] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[i][e], h[i][e], av[e % NA], 0, 0, 0);
            au[e % NA] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[i][e], h[i][e], au[e % NA], 0, 0, 0);
          }
        }
    }
    float* mine = red + wave * 32 * 64 + lane;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      mine[r * 64] = BWD ? av[0][r] + av[NA - 1][r] : av[0][r];
      mine[(16 + r) * 64] = BWD ? au[0][r] + au[NA - 1][r] : au[0][r];
    }
    if constexpr (BWD) aux[wave * 64 + lane] = dot;
    __syncthreads();
    if (wave < 4) {   // wavefront q: gate units q * 8 + half * 4 .. + 3 of the block, row li
      const int j0 = ub * 32 + wave * 8 + half * 4;
      float xv[4] = {0.f, 0.f, 0.f, 0.f}, xu[4] = {0.f, 0.f, 0.f, 0.f};
      for (int w = 0; w < W; w += 4)   // W is 4 or 8
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float* q = red + (w * 32 + wave * 4 + e) * 64 + lane;
          xv[e] += (q[0] + q[32 * 64]) + (q[64 * 64] + q[96 * 64]);
          q += 16 * 64;
          xu[e] += (q[0] + q[32 * 64]) + (q[64 * 64] + q[96 * 64]);
        }
      float da = 0.f;
      if constexpr (BWD) {
        for (int w = 0; w < W; w += 4) {   // short chains: what the rows' dot products are off by adds up over the rows
          float t[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) t[i] = aux[(w + i) * 64 + li] + aux[(w + i) * 64 + 32 + li];
          da += (t[0] + t[1]) + (t[2] + t[3]);
        }
        da = ok ? da * (__expf(p.a[n] - p.scal[0]) / p.scal[1]) : 0.f;
      }
      float dv[4], du[4], dw[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = j0 + e < Mh ? j0 + e : Mh - 1;
        const float t = tanhf(xv[e] + p.Vb[j]), s = 1.0f / (1.0f + __expf(-(xu[e] + p.Ub[j]))), wj = p.w[j];
        if constexpr (BWD) {
          dv[e] = da * wj * s * (1.f - t * t);
          du[e] = da * wj * t * s * (1.f - s);
          dw[e] = da * t * s;
        } else if (j0 + e < Mh) {
          part += wj * t * s;
        }
      }
      if constexpr (BWD) {
        float* row = out + n * 2 * Mh + j0;
        if (ok) {
          if (VEC && j0 < Mh) {
            *reinterpret_cast<f32x4*>(row) = f32x4{dv[0], dv[1], dv[2], dv[3]};
            *reinterpret_cast<f32x4*>(row + Mh) = f32x4{du[0], du[1], du[2], du[3]};
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (j0 + e < Mh) { row[e] = dv[e]; row[Mh + e] = du[e]; }
          }
        }
#pragma unroll
        for (int o = 1; o < 32; o <<= 1)
#pragma unroll
          for (int e = 0; e < 4; ++e) dw[e] += __shfl_xor(dw[e], o, 64);
        if (li == 0) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (j0 + e < Mh) dwp[(size_t)blockIdx.x * Mh + j0 + e] = dw[e];
        }
      }
    }
    if constexpr (!BWD) {
      if (wave < 4) aux[wave * 64 + lane] = part;
    }
    __syncthreads();   // the partial blocks have been read
    if constexpr (!BWD) {   // (aux is next written behind the next block's barrier)
      if (threadIdx.x < 32) {
        float a = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q) a += aux[q * 64 + li] + aux[q * 64 + 32 + li];
        logit += a;
      }
    }
  }
  if constexpr (!BWD) {
    if (threadIdx.x < 32 && ok) out[blockIdx.y * p.N + n] = logit;
  }
}

// Attention logits from their `parts` partial sums (part[i][n]), and per workgroup {max, sum, weighted feature sum} over
// its groups of GR rows (the weighted sum in fp64: it feeds a cancelling difference in the backward).
// WIDE: part[n] holds the row's [t | s] (2 M_h) instead, and the logit is summed over the gate units here, in order.
template <int GR, bool WIDE>
__global__ void __launch_bounds__(256) pool_softmax_part_k(PoolArgs p, const float* __restrict__ part, int parts) {
  extern __shared__ double zb[];   // [D]
  __shared__ float er[GR];
  __shared__ float resc;
  const int D = p.D, tid = threadIdx.x;
  for (int d = tid; d < D; d += 256) zb[d] = 0.0;
  float m = -INFINITY;   // of the rows so far
  double l = 0.0;
  const long long groups = (p.N + GR - 1) / GR;
  for (long long g = blockIdx.x; g < groups; g += gridDim.x) {
    const long long n0 = g * GR;
    if (tid < GR) {
      float a = -INFINITY;
      if (n0 + tid < p.N) {
        a = 0.f;
        if constexpr (WIDE) {
          const int Mh = p.Mh;
          const float* ts = part + (n0 + tid) * 2 * Mh;
#pragma unroll 8
          for (int j = 0; j < Mh; ++j) a += p.w[j] * ts[j] * ts[Mh + j];
        } else {
          for (int i = 0; i < parts; ++i) a += part[i * p.N + n0 + tid];
        }
        p.a[n0 + tid] = a;
      }
      float mx = a;
#pragma unroll
      for (int o = GR / 2; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, GR));
      mx = fmaxf(m, mx);
      const float sc = __expf(m - mx), e = __expf(a - mx);   // exp(-inf) = 0 on the first group
      double es = (double)e;
#pragma unroll
      for (int o = GR / 2; o > 0; o >>= 1) es += __shfl_xor(es, o, GR);
      l = l * (double)sc + es;
      m = mx;
      er[tid] = e;
      if (tid == 0) resc = sc;
    }
    __syncthreads();
    const double sc = (double)resc;
    for (int d = tid; d < D; d += 256) {
      const float* h = p.H + n0 * D + d;
      float v[GR];
#pragma unroll
      for (int r = 0; r < GR; ++r) v[r] = h[(n0 + r < p.N ? r : 0) * (long long)D];
      double z = zb[d] * sc;
#pragma unroll
      for (int r = 0; r < GR; ++r) z += (double)er[r] * (double)v[r];   // rows past the end have weight zero
      zb[d] = z;
    }
    __syncthreads();
  }
  double* out = p.part + (size_t)blockIdx.x * (2 + D);
  if (tid == 0) { out[0] = (double)m; out[1] = l; }
  for (int d = tid; d < D; d += 256) out[2 + d] = zb[d];
}

// G[n][d] = alpha_n dz[d] + sum_j Dp[n][j] [V;U][j][d]: 32 rows x 32 features per workgroup, gate units split over four
// wavefronts
constexpr int UG = 4;
template <bool VEC>
__global__ void __launch_bounds__(256) pool_g_f32_k(PoolArgs p, const float* __restrict__ Dp) {
  __shared__ float red[4][16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 31, half = lane >> 5;
  const int D = p.D, Mh = p.Mh, K = 2 * Mh, nc = (K + 7) / 8;
  const long long n = (long long)blockIdx.x * 32 + li;
  const bool ok = n < p.N;
  const int d = blockIdx.y * 32 + li, dc = d < D ? d : D - 1;
  const float* drow = Dp + (ok ? n : p.N - 1) * K;
  pool_head_grads(p);
  f32x16 acc = zero16();
  for (int c0 = wave; c0 < nc; c0 += 4 * UG) {
    f32x4 g[UG];
    float w[UG][4];
#pragma unroll
    for (int i = 0; i < UG; ++i) {
      const int j0 = (c0 + i * 4) * 8 + half * 4;
      g[i] = ld4<VEC>(drow, j0, K);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = j0 + e < K ? j0 + e : K - 1;   // its factor is zero
        w[i][e] = (j < Mh ? p.VW + (size_t)j * D : p.UW + (size_t)(j - Mh) * D)[dc];
      }
    }
#pragma unroll
    for (int i = 0; i < UG; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(w[i][e], g[i][e], acc, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) red[wave][r][lane] = acc[r];
  __syncthreads();
  if (!ok) return;
  const float alpha = __expf(p.a[n] - p.scal[0]) / p.scal[1];
  const float* dz = p.scal + pool_z_off(p.C) + D;
  const int d0 = blockIdx.y * 32 + wave * 8 + half * 4;
  f32x4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int r = wave * 4 + e;
    v[e] = alpha * dz[d0 + e < D ? d0 + e : D - 1] + ((red[0][r][lane] + red[1][r][lane]) + (red[2][r][lane] + red[3][r][lane]));
  }
  float* o = p.G + n * D + d0;
  if constexpr (VEC) {
    if (d0 < D) *reinterpret_cast<f32x4*>(o) = v;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (d0 + e < D) o[e] = v[e];
  }
}

// ---- backward of long bags ----
// The same two products on the bf16 matrix cores, operands cut into three bf16 terms (split_f32.h): 64 rows x 64 gate units
// (features) per workgroup.  What bounds it: the six products' MFMAs (0.75 PFLOP/s of bf16 at 131,072 rows) beside the cut of the
// operands and the fragments' trips from LDS.  The products of the leading terms have an accumulator of their own: the gate gradients' terms
// cancel, and what a sum is off by is mostly the roundings of its additions, of which six products a step in one
// accumulator would make six times as many.  A row's dot product with dz is added in 64 bits, and the low part of z goes into it as a sum of its own:
// taken off the differences h - z, which lie on a coarse grid, it would be rounded the same way in every row, and the gate units' sums over
// the rows, which cancel, would show that.  (Errors against 64 bits over those of the kernels above, geometric means over bags of 8,192 to 65,536
// rows, D = 384, M_h = 128: V.W 0.84, b_V 0.81, U.W 0.85, b_U 0.85, w 0.92.)
// us, before / now, D = 768: 45,056 rows, M_h = 128: gates 421 / 145, G 293 / 140; whole step of 131,072 rows 3092 / 1352, M_h = 256
// 6340 / 2400.  (128 x 128 results a workgroup: 151 and 133, nothing either way.)
constexpr int NACC = 2;   // accumulators of a block
constexpr int SBM = 64, SPB = 128;   // rows; columns of the second operand: 64 units of V and of U, or 128 features

// acc[j][0] the leading products, acc[j][1] the others; blocks j are 32 rows of B
__device__ __forceinline__ void split_mul(const bf16* s, int oa, int ob, int half, f32x16 (&acc)[2][NACC]) {
#pragma unroll
  for (int ks = 0; ks < SPLIT_BK / 16; ++ks) {
    const Split fa = get_split<SBM + SPB>(s, oa, ks * 2 + half);
    Split fb[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) fb[j] = get_split<SBM + SPB>(s, ob + j * 32, ks * 2 + half);
#pragma unroll
    for (int t = 0; t < 6; ++t)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        f32x16& c = acc[j][t < 5];
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j].t[TERM_B[t]], fa.t[TERM_A[t]], c, 0, 0, 0);
      }
  }
}
// row panels are dealt to the XCDs, a panel's column tiles to one: false past the end
__device__ __forceinline__ bool split_tile(int MT, int NT, int& mt, int& nt) {
  const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
  mt = (slot / NT) * 8 + xcd;
  nt = slot % NT;
  return mt < MT;
}

// pool_gate_f32_k<true, true> by tiles: Dp, and dwp[2 mt + i][j] the sums over 32 rows.  D a multiple of 32, M_h of 64.
__global__ void __launch_bounds__(256, 3) pool_dgate_split_k(PoolArgs p, float* __restrict__ Dp, float* __restrict__ dwp, int MT, int NT) {
  constexpr int ROWS = SBM + SPB;
  __shared__ __attribute__((aligned(16))) bf16 st[3 * ROWS * SPLIT_BK];
  __shared__ float da[SBM];
  extern __shared__ __attribute__((aligned(16))) float zc[];   // [3][D]: z, dz, the rest of z
  int mt, nt;
  if (!split_tile(MT, NT, mt, nt)) return;
  const int D = p.D, Mh = p.Mh, nk = D / SPLIT_BK;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int frow = lane & 31, half = lane >> 5, wm = wave >> 1, wn = wave & 1;
  const long long m0 = (long long)mt * SBM;
  for (int i = tid; i < 3 * D; i += 256) zc[i] = p.scal[pool_z_off(p.C) + i];
  // the loader's rows: one of H (past the end the last one, never stored), then row tid / 4 of two blocks of 64: 32 gate units of V and the
  // same of U each, so that a wavefront's two blocks belong together
  const int lr = tid >> 2, lc = (tid & 3) * 8;
  const float* src[3];
  src[0] = p.H + (m0 + lr < p.N ? m0 + lr : p.N - 1) * D + lc;
#pragma unroll
  for (int j = 0; j < 2; ++j) src[1 + j] = (lr < 32 ? p.VW : p.UW) + (size_t)(nt * 64 + j * 32 + (lr & 31)) * D + lc;
  f32x4 x[3][2];
  auto load = [&](int kt) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      x[j][0] = *reinterpret_cast<const f32x4*>(src[j] + kt * SPLIT_BK);
      x[j][1] = *reinterpret_cast<const f32x4*>(src[j] + kt * SPLIT_BK + 4);
    }
  };
  f32x16 acc[2][NACC];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < NACC; ++i) acc[j][i] = zero16();
  double dot = 0.0;   // (64 bits: what it is off by goes into every gate unit's gradient)
  const int oa = wm * 32 + frow, ob = SBM + wn * 64 + frow;
  load(0);
  for (int kt = 0; kt < nk; ++kt) {
    step_barrier();   // every wavefront is done with the step before (the first: the columns of z are there)
#pragma unroll
    for (int j = 0; j < 3; ++j) put_split<ROWS>(st, j * 64 + lr, tid & 3, split_of(x[j][0], x[j][1]));
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const float* c = zc + kt * SPLIT_BK + lc + q * 4;
      const f32x4 z = *reinterpret_cast<const f32x4*>(c), dz = *reinterpret_cast<const f32x4*>(c + D), zl = *reinterpret_cast<const f32x4*>(c + 2 * D);
      const f32x4 t = (x[0][q] - z) * dz, l = zl * dz;
      dot += (double)((t[0] + t[1]) + (t[2] + t[3])) - (double)((l[0] + l[1]) + (l[2] + l[3]));
    }
    if (kt + 1 < nk) load(kt + 1);
    step_barrier();
    split_mul(st, oa, ob, half, acc);
  }
  {
    dot += __shfl_xor(dot, 1, 64);
    dot += __shfl_xor(dot, 2, 64);
    const long long n = m0 + lr;
    if ((tid & 3) == 0) da[lr] = n < p.N ? (float)dot * (__expf(p.a[n] - p.scal[0]) / p.scal[1]) : 0.f;
  }
  f32x16 r[2][1];
#pragma unroll
  for (int j = 0; j < 2; ++j) r[j][0] = acc[j][0] + acc[j][1];
  if (not_finite(r)) {   // (an infinite feature or weight has an infinite product, not none: in float32)
    const long long n = m0 + oa < p.N ? m0 + oa : p.N - 1;
    const float* ph = p.H + n * D + half * 4;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const float* pw = (j ? p.UW : p.VW) + (size_t)(nt * 64 + wn * 32 + frow) * D + half * 4;
      r[j][0] = zero16();
#pragma nounroll
      for (int k = 0; k < D; k += 8) {
        const f32x4 u = *reinterpret_cast<const f32x4*>(ph + k), v = *reinterpret_cast<const f32x4*>(pw + k);
#pragma unroll
        for (int e = 0; e < 4; ++e) r[j][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[e], u[e], r[j][0], 0, 0, 0);
      }
    }
  }
  __syncthreads();
  const long long n = m0 + oa;
  const bool ok = n < p.N;
  const float g = da[oa];
  float* row = Dp + n * 2 * Mh;
  float* dwrow = dwp + (size_t)(2 * mt + wm) * Mh;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int j0 = nt * 64 + wn * 32 + q * 8 + half * 4;
    f32x4 dv, du;
    float dw[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int j = j0 + e;
      const float t = tanhf(r[0][0][q * 4 + e] + p.Vb[j]), s = 1.0f / (1.0f + __expf(-(r[1][0][q * 4 + e] + p.Ub[j]))), wj = p.w[j];
      dv[e] = g * wj * s * (1.f - t * t);
      du[e] = g * wj * t * s * (1.f - s);
      dw[e] = g * t * s;
    }
    if (ok) {
      *reinterpret_cast<f32x4*>(row + j0) = dv;
      *reinterpret_cast<f32x4*>(row + Mh + j0) = du;
    }
#pragma unroll
    for (int o = 1; o < 32; o <<= 1)
#pragma unroll
      for (int e = 0; e < 4; ++e) dw[e] += __shfl_xor(dw[e], o, 64);
    if (frow == 0 && m0 + wm * 32 < p.N) *reinterpret_cast<f32x4*>(dwrow + j0) = f32x4{dw[0], dw[1], dw[2], dw[3]};
  }
}

// pool_g_f32_k by tiles of 64 rows x 128 features
__global__ void __launch_bounds__(256, 3) pool_g_split_k(PoolArgs p, const float* __restrict__ Dp, int MT, int NT) {
  constexpr int ROWS = SBM + SPB;
  __shared__ __attribute__((aligned(16))) bf16 st[3 * ROWS * SPLIT_BK];
  pool_head_grads(p);
  int mt, nt;
  if (!split_tile(MT, NT, mt, nt)) return;
  const int D = p.D, Mh = p.Mh, K = 2 * Mh, nk = K / SPLIT_BK;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int frow = lane & 31, half = lane >> 5, wm = wave >> 1, wn = wave & 1;
  const long long m0 = (long long)mt * SBM;
  const int d0 = nt * SPB;
  // the weights' rows are the contracted index here: a lane loads eight of them at its feature
  const int lr = tid >> 2, lc = (tid & 3) * 8;
  const float* ha = Dp + (m0 + lr < p.N ? m0 + lr : p.N - 1) * K + lc;
  int dc[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) dc[j] = d0 + j * 64 + lane < D ? d0 + j * 64 + lane : D - 1;
  f32x4 x[2];
  float w[2][8];
  auto load = [&](int kt) __attribute__((always_inline)) {
    x[0] = *reinterpret_cast<const f32x4*>(ha + kt * SPLIT_BK);
    x[1] = *reinterpret_cast<const f32x4*>(ha + kt * SPLIT_BK + 4);
    const int j0 = kt * SPLIT_BK + wave * 8;
    const float* wr = j0 < Mh ? p.VW + (size_t)j0 * D : p.UW + (size_t)(j0 - Mh) * D;   // M_h is a multiple of 64
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 8; ++e) w[j][e] = wr[(size_t)e * D + dc[j]];
  };
  f32x16 acc[2][NACC];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < NACC; ++i) acc[j][i] = zero16();
  const int oa = wm * 32 + frow, ob = SBM + wn * 64 + frow;
  load(0);
  for (int kt = 0; kt < nk; ++kt) {
    if (kt) step_barrier();   // every wavefront is done with the step before
    put_split<ROWS>(st, lr, tid & 3, split_of(x[0], x[1], SPLIT_UP));
#pragma unroll
    for (int j = 0; j < 2; ++j) put_split<ROWS>(st, SBM + j * 64 + lane, wave, split8(w[j]));
    if (kt + 1 < nk) load(kt + 1);
    step_barrier();
    split_mul(st, oa, ob, half, acc);
  }
  f32x16 r[2][1];
#pragma unroll
  for (int j = 0; j < 2; ++j) r[j][0] = acc[j][0] + acc[j][1];
  const long long n = m0 + oa < p.N ? m0 + oa : p.N - 1;
  if (!not_finite(r)) {
    scale_down(r, SPLIT_UP);
  } else {
    const float* pd = Dp + n * K + half * 4;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int d = d0 + wn * 64 + j * 32 + frow < D ? d0 + wn * 64 + j * 32 + frow : D - 1;
      r[j][0] = zero16();
#pragma nounroll
      for (int k = 0; k < K; k += 8) {
        const f32x4 u = *reinterpret_cast<const f32x4*>(pd + k);
        const int j0 = k + half * 4;
        const float* wr = (j0 < Mh ? p.VW + (size_t)j0 * D : p.UW + (size_t)(j0 - Mh) * D) + d;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[j][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(wr[(size_t)e * D], u[e], r[j][0], 0, 0, 0);
      }
    }
  }
  if (m0 + oa >= p.N) return;
  const float alpha = __expf(p.a[n] - p.scal[0]) / p.scal[1];
  const float* dz = p.scal + pool_z_off(p.C) + D;
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int d = d0 + wn * 64 + j * 32 + q * 8 + half * 4;
      if (d >= D) continue;
      const f32x16& v = r[j][0];
      const f32x4 z = {dz[d], dz[d + 1], dz[d + 2], dz[d + 3]};
      *reinterpret_cast<f32x4*>(p.G + n * D + d) = alpha * z + f32x4{v[q * 4], v[q * 4 + 1], v[q * 4 + 2], v[q * 4 + 3]};
    }
}

// ---- wide rows ----
// D > 1536 is the feature row of a bottleneck encoder (2048).  The gradient that leaves here runs back through some fifty
// batch-normalised layers whose parameter gradients are sums of terms that cancel: the last bit of G decides bf16 roundings all the
// way down and moves them by 1.5 %.  So there every sum keeps one order whatever the shape: a dot product over D is one
// wavefront's, lane l taking d = l, l + 64, ..., sums over the gate units run in order in one thread.  What is free is cut:
// gate units over workgroups (all of them in one workgroup per 8 rows: 300 x 2048, M_h = 128 682 us forward, 1032 backward).
constexpr int WR = 8;    // rows per workgroup: 64 KB of features
bool wide(const PoolArgs& p) { return p.D > 1536; }

// TS[n] = [tanh(V h + b_V) | sigmoid(U h + b_U)]
__global__ void __launch_bounds__(256) pool_wide_gate_k(PoolArgs p, float* __restrict__ TS) {
  extern __shared__ float hs[];   // [WR][D]
  const int D = p.D, Mh = p.Mh, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long n0 = (long long)blockIdx.x * WR;
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *p.ticket = 0;
#pragma unroll
  for (int r = 0; r < WR; ++r)
    for (int d = threadIdx.x; d < D; d += 256) hs[r * D + d] = n0 + r < p.N ? p.H[(n0 + r) * D + d] : 0.f;
  __syncthreads();
  for (int j = blockIdx.y * 4 + wave; j < Mh; j += gridDim.y * 4) {
    const float *vr = p.VW + (size_t)j * D, *ur = p.UW + (size_t)j * D;
    float av[WR], au[WR];
#pragma unroll
    for (int r = 0; r < WR; ++r) av[r] = au[r] = 0.f;
#pragma unroll 8
    for (int d = lane; d < D; d += 64) {
      const float v = vr[d], u = ur[d];
#pragma unroll
      for (int r = 0; r < WR; ++r) {
        const float h = hs[r * D + d];
        av[r] += v * h;
        au[r] += u * h;
      }
    }
#pragma unroll
    for (int r = 0; r < WR; ++r) {
      av[r] = wave_sum(av[r]);
      au[r] = wave_sum(au[r]);
    }
    if (lane == 0) {
      const float bv = p.Vb[j], bu = p.Ub[j];
#pragma unroll
      for (int r = 0; r < WR; ++r)
        if (n0 + r < p.N) {
          TS[(n0 + r) * 2 * Mh + j] = tanhf(av[r] + bv);
          TS[(n0 + r) * 2 * Mh + Mh + j] = 1.0f / (1.0f + __expf(-(au[r] + bu)));
        }
    }
  }
}

// [t | s] of 32 rows -> [dpV | dpU] in place, dwp[blockIdx.x][j] = sum over the rows of da t s
__global__ void __launch_bounds__(512) pool_wide_dgate_k(PoolArgs p, float* __restrict__ TS, float* __restrict__ dwp) {
  __shared__ float da[32];
  const int D = p.D, Mh = p.Mh, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long n0 = (long long)blockIdx.x * 32;
  const float* zv = p.scal + pool_z_off(p.C);
  for (int r = wave; r < 32; r += 8) {   // softmax backward: da_n = alpha_n (h_n - z) . dz
    const bool ok = n0 + r < p.N;
    const float* h = p.H + (ok ? n0 + r : p.N - 1) * D;
    float acc = 0.f;
#pragma unroll 8
    for (int d = lane; d < D; d += 64) acc += ((h[d] - zv[d]) - zv[2 * D + d]) * zv[D + d];
    acc = wave_sum(acc);
    if (lane == 0) {
      const float a = ok ? __expf(p.a[n0 + r] - p.scal[0]) / p.scal[1] : 0.f;
      da[r] = a * acc;
    }
  }
  __syncthreads();
  const int rows = p.N - n0 < 32 ? (int)(p.N - n0) : 32;
  for (int j = threadIdx.x; j < Mh; j += 512) {
    const float wj = p.w[j];
    float dw = 0.f;
#pragma unroll 4
    for (int r = 0; r < rows; ++r) {
      float* row = TS + (n0 + r) * 2 * Mh;
      const float t = row[j], s = row[Mh + j], g = da[r];
      const float dv = g * wj * s * (1.f - t * t);
      const float du = g * wj * t * s * (1.f - s);
      row[j] = dv;
      row[Mh + j] = du;
      dw += g * t * s;
    }
    dwp[(size_t)blockIdx.x * Mh + j] = dw;
  }
}

// G[n][d] = alpha_n dz[d] + sum_j dpV[n][j] V[j][d] + dpU[n][j] U[j][d]: 8 rows x 256 features per workgroup
__global__ void __launch_bounds__(256) pool_wide_g_k(PoolArgs p, const float* __restrict__ Dp) {
  extern __shared__ float dl[];   // [WR][2 Mh]
  const int D = p.D, Mh = p.Mh;
  const long long n0 = (long long)blockIdx.x * WR;
  pool_head_grads(p);
  for (int i = threadIdx.x; i < WR * 2 * Mh; i += 256) dl[i] = n0 * 2 * Mh + i < p.N * 2 * Mh ? Dp[n0 * 2 * Mh + i] : 0.f;
  __syncthreads();
  const int d = blockIdx.y * 256 + threadIdx.x;
  if (d >= D) return;
  const float dzd = p.scal[pool_z_off(p.C) + D + d];
  float acc[WR];
#pragma unroll
  for (int r = 0; r < WR; ++r) {
    const float al = n0 + r < p.N ? __expf(p.a[n0 + r] - p.scal[0]) / p.scal[1] : 0.f;
    acc[r] = al * dzd;
  }
#pragma unroll 8
  for (int j = 0; j < Mh; ++j) {
    const float v = p.VW[(size_t)j * D + d], u = p.UW[(size_t)j * D + d];
#pragma unroll
    for (int r = 0; r < WR; ++r) acc[r] += dl[r * 2 * Mh + j] * v + dl[r * 2 * Mh + Mh + j] * u;
  }
#pragma unroll
  for (int r = 0; r < WR; ++r)
    if (n0 + r < p.N) p.G[(n0 + r) * D + d] = acc[r];
}

// 16-byte accesses to rows of D features and of M_h gate units
bool vec_ok(const PoolArgs& p) {
  auto al = [](const void* q) { return ((uintptr_t)q & 15) == 0; };
  return p.D % 4 == 0 && p.Mh % 4 == 0 && al(p.H) && al(p.VW) && al(p.UW) && (!p.G || al(p.G));
}

// Wavefronts that share a contraction over D: about six steps of eight each, all of whose loads a wavefront keeps in flight.
int gate_waves(int D) { return D <= 256 ? 4 : 8; }
size_t gate_lds(int W) { return (size_t)W * 33 * 64 * sizeof(float); }

template <bool VEC, bool BWD>
hipError_t go_gate(const PoolArgs& p, float* out, float* dwp, int parts, hipStream_t s) {
  const int W = gate_waves(p.D);
  auto kern = pool_gate_f32_k<VEC, BWD>;
  if (gate_lds(W) > 65536) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)gate_lds(W));
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)((p.N + 31) / 32), parts), dim3(64 * W), gate_lds(W), s, p, out, dwp);
  return hipGetLastError();
}

hipError_t go_wide_gate(const PoolArgs& p, float* TS, hipStream_t s) {
  // gate units over as many workgroups as make about four rounds of the chip
  const long long groups = (p.N + WR - 1) / WR;
  const int most = (p.Mh + 3) / 4;
  long long ny = (1024 + groups - 1) / groups;
  if (ny > most) ny = most;
  hipLaunchKernelGGL(pool_wide_gate_k, dim3((unsigned)groups, (unsigned)ny), dim3(256), (size_t)WR * p.D * 4, s, p, TS);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_pool_softmax_part(const PoolArgs& p, const float* part, int parts, hipStream_t s) {
  hipLaunchKernelGGL((pool_softmax_part_k<16, false>), dim3(p.blocks), dim3(256), (size_t)p.D * 8, s, p, part, parts);
  return hipGetLastError();
}

hipError_t launch_pool_gate_part_f32(const PoolArgs& p, hipStream_t s) {
  if (wide(p)) {
    if ((size_t)p.N * 2 * p.Mh > p.a_room) return hipErrorInvalidValue;
    hipError_t e = go_wide_gate(p, p.a_tmp, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((pool_softmax_part_k<WR, true>), dim3(p.blocks), dim3(256), (size_t)p.D * 8, s, p, p.a_tmp, 0);
    return hipGetLastError();
  }
  int parts = (p.Mh + 31) / 32;
  if ((size_t)parts * p.N > p.a_room) parts = 1;   // the fixed array of mil_pool_fwd_static, near its limit
  if ((size_t)p.N > p.a_room) return hipErrorInvalidValue;
  hipError_t e = vec_ok(p) ? go_gate<true, false>(p, p.a_tmp, nullptr, parts, s) : go_gate<false, false>(p, p.a_tmp, nullptr, parts, s);
  if (e != hipSuccess) return e;
  return launch_pool_softmax_part(p, p.a_tmp, parts, s);
}

// Dp: [N][2 M_h]; dwp: [ceil(N / 32)][M_h] partial sums of dw; writes p.G and the head's gradients
// By tiles where the gates make more than 128 of them, half the chip: at 128 (4,096 rows, M_h = 128) both take 146 us for a step, at 256 it is
// 225 / 166, at 32 106 / 134 (a tile is a chain of D / 32 steps, which the kernels above deal to their wavefronts).
constexpr long long SPLIT_TILES = 128;
hipError_t launch_pool_bwd_f32(const PoolArgs& p, float* Dp, float* dwp, hipStream_t s) {
  if (wide(p)) {
    // t and s once more: an earlier backward over the same forward has written over them
    hipError_t e = go_wide_gate(p, Dp, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(pool_wide_dgate_k, dim3((unsigned)((p.N + 31) / 32)), dim3(512), 0, s, p, Dp, dwp);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(pool_wide_g_k, dim3((unsigned)((p.N + WR - 1) / WR), (p.D + 255) / 256), dim3(256),
                       (size_t)WR * 2 * p.Mh * 4, s, p, Dp);
    return hipGetLastError();
  }
  const int parts = (p.Mh + 31) / 32;
  const bool vec = vec_ok(p);
  if (vec && ((p.N + SBM - 1) / SBM) * (p.Mh / 64) > SPLIT_TILES && p.N < (1LL << 31) && p.D % SPLIT_BK == 0 && p.Mh % 64 == 0) {
    const int MT = (int)((p.N + SBM - 1) / SBM), NTu = p.Mh / 64, NTd = (p.D + SPB - 1) / SPB;
    const long long panels = (MT + 7) / 8 * 8;
    hipLaunchKernelGGL(pool_dgate_split_k, dim3((unsigned)(panels * NTu)), dim3(256), (size_t)3 * p.D * 4, s, p, Dp, dwp, MT, NTu);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(pool_g_split_k, dim3((unsigned)(panels * NTd)), dim3(256), 0, s, p, Dp, MT, NTd);
    return hipGetLastError();
  }
  hipError_t e = vec ? go_gate<true, true>(p, Dp, dwp, parts, s) : go_gate<false, true>(p, Dp, dwp, parts, s);
  if (e != hipSuccess) return e;
  const dim3 grid((unsigned)((p.N + 31) / 32), (p.D + 31) / 32);
  if (vec) hipLaunchKernelGGL(pool_g_f32_k<true>, grid, dim3(256), 0, s, p, Dp);
  else hipLaunchKernelGGL(pool_g_f32_k<false>, grid, dim3(256), 0, s, p, Dp);
  return hipGetLastError();
}

}  // namespace sl
