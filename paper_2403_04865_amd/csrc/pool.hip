// Gated-attention MIL pooling over the tile features of a slide, forward and backward.
//   t_n = tanh(V h_n + b_V), s_n = sigmoid(U h_n + b_U), a_n = w . (t_n * s_n),
//   alpha = softmax_n(a), z = sum_n alpha_n h_n, y = W_c z + b_c, loss = BCE / CE(y, label).
// The softmax over tiles is a two-level online reduction: every workgroup of stage 1 (pool_mfma.hip, pool_f32.hip) keeps a
// running (max, sum, weighted feature sum) over its row groups, stage 2 combines them.
#include "slide_internal.h"

namespace sl {

// Softmax statistics over the partials of stage 1: running max m and normaliser Z of the whole slide; wts[b] is
// the weight exp(m_b - m) of partial b.  Called by all 256 threads of a workgroup.
__device__ void pool_partial_stats(const PoolArgs& p, float* sm, double* smd, float* wts, float& m_out, double& Z_out) {
  const int D = p.D, B = p.blocks, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  float bm[4];   // at most 1024 partials
  double bl[4];
  float m = -INFINITY;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int b = threadIdx.x + i * 256;
    const double* q = p.part + (size_t)(b < B ? b : 0) * (2 + D);
    bm[i] = b < B ? (float)q[0] : -INFINITY;
    bl[i] = q[1];
    m = fmaxf(m, bm[i]);
  }
  m = wave_max(m);
  if (lane == 0) sm[w] = m;
  __syncthreads();
  m = fmaxf(fmaxf(sm[0], sm[1]), fmaxf(sm[2], sm[3]));
  double l = 0.0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int b = threadIdx.x + i * 256;
    const float wt = __expf(bm[i] - m);   // 0 past the last partial
    if (b < B) {
      wts[b] = wt;
      l += bl[i] * (double)wt;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o, 64);
  if (lane == 0) smd[w] = l;
  __syncthreads();
  m_out = m;
  Z_out = (smd[0] + smd[1]) + (smd[2] + smd[3]);
}

// forward, stage 2: z, softmax weights, logits, loss and the head's gradients in one launch.
//   workgroups 0 .. nz - 1: z = sum_b wts[b] z_b / Z, 16 columns each, 16 slices of the partials per column: a single
//     compute unit fetching all partials (written by every other unit a moment ago) is bound by its own handful of
//     outstanding misses, so the sum is spread over D / 16 units with every load of a thread in flight at once;
//   the others: alpha, 1,024 rows each;
//   whichever z workgroup finishes last (a counter that stage 1 clears) goes on with m, Z, logits, loss, dy, dz, z.dz: on a
//     bag of a few dozen rows each further launch costs as much as all of the arithmetic.
__global__ void __launch_bounds__(256) pool_combine_k(PoolArgs p, int nz) {
  __shared__ float sm[256];
  __shared__ double smd[256];
  __shared__ float wts[1024];   // at most 1024 workgroups in stage 1
  __shared__ double red[16][17];
  __shared__ int last;
  __shared__ float zs[2048];    // at most 2048 features
  const int D = p.D, C = p.C, B = p.blocks;
  float* scal = p.scal;
  float* y = scal + 4;
  float* dy = y + C;
  float* z = scal + pool_z_off(C);
  float* dz = z + D;
  float* zlo = dz + D;
  float m;
  double Z;
  // a chain of trips to memory bounds this kernel, so what it will need is asked for at its start: this thread's partials (up to 256
  // workgroups: 16 of them) and, for whoever comes last, this wavefront's first class of the head.  Not for a few partials: on 16
  // tiles of the two-block encoder these 24 loads whatever the sizes made the kernel 0.7 us slower (1,037 rows: 1.1 us faster)
  const bool early = B > 16;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int c16 = threadIdx.x & 15, sl = threadIdx.x >> 4;
  const int d16 = (int)blockIdx.x * 16 + c16, dc = d16 < D ? d16 : D - 1;
  double pv[16];
  float cw[8];
  float cb0 = 0.f;
  if (early && (int)blockIdx.x < nz) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int b = sl + 16 * i;
      pv[i] = p.part[(size_t)(b < B ? b : 0) * (2 + D) + 2 + dc];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int d = lane + 64 * i;
      cw[i] = p.cW[(size_t)(w < C ? w : 0) * D + (d < D ? d : 0)];
    }
    cb0 = p.cb[w < C ? w : 0];
  }
  pool_partial_stats(p, sm, smd, wts, m, Z);
  if ((int)blockIdx.x >= nz) {
    const float Zf = (float)Z;
    for (long long i = (long long)(blockIdx.x - nz) * 1024 + threadIdx.x, k = 0; k < 4; ++k, i += 256)
      if (i < p.N) p.alpha[i] = __expf(p.a[i] - m) / Zf;
    return;
  }
  {
    const int c = c16, d = d16;
    double acc = 0.0;
    if (early) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (sl + 16 * i < B) acc += pv[i] * (double)wts[sl + 16 * i];
    }
#pragma unroll 8
    for (int b = early ? sl + 256 : sl; b < B; b += 16) acc += p.part[(size_t)b * (2 + D) + 2 + dc] * (double)wts[b];
    red[sl][c] = acc;
    __syncthreads();
    if (threadIdx.x < 16 && d < D) {
      double t = 0.0;
#pragma unroll
      for (int i = 0; i < 16; ++i) t += red[i][c];
      t /= Z;
      float hi = (float)t;
      // z = z[d] + zlo[d] to fp64 accuracy; stored past this die's L2 for whichever workgroup comes last
      __hip_atomic_store(z + d, hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(zlo + d, (float)(t - (double)hi), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (threadIdx.x < 64) {   // the wavefront that stored them: they have arrived before the ticket is drawn
      __builtin_amdgcn_s_waitcnt(0);
      asm volatile("" ::: "memory");
      if (threadIdx.x == 0) last = __hip_atomic_fetch_add(p.ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)nz - 1;
    }
    __syncthreads();
    if (!last) return;
    for (int i = threadIdx.x; i < D; i += 256) zs[i] = __hip_atomic_load(z + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
  }
  // logits: one wave per class round-robin
  for (int c = w; c < C; c += 4) {
    float acc = 0.f;
    const bool have = early && c == w;
    if (have) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (lane + 64 * i < D) acc += cw[i] * zs[lane + 64 * i];
    }
    for (int d = have ? lane + 512 : lane; d < D; d += 64) acc += p.cW[(size_t)c * D + d] * zs[d];
    acc = wave_sum(acc);
    if (lane == 0) y[c] = acc + (have ? cb0 : p.cb[c]);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float loss;
    if (C == 1) {
      float v = y[0];
      loss = fmaxf(v, 0.f) - v * (float)p.label + log1pf(__expf(-fabsf(v)));
      dy[0] = 1.0f / (1.0f + __expf(-v)) - (float)p.label;
    } else {
      float mx = y[0];
      for (int c = 1; c < C; ++c) mx = fmaxf(mx, y[c]);
      float se = 0.f;
      for (int c = 0; c < C; ++c) se += __expf(y[c] - mx);
      float lse = mx + logf(se);
      loss = lse - y[p.label];
      for (int c = 0; c < C; ++c) dy[c] = __expf(y[c] - lse) - (c == p.label ? 1.f : 0.f);
    }
    scal[0] = m; scal[1] = (float)Z; scal[2] = loss;
    if (p.loss) p.loss[0] = loss;
    if (p.logits) for (int c = 0; c < C; ++c) p.logits[c] = y[c];
  }
  if (p.fwd_only) return;
  __syncthreads();
  float part = 0.f;
  for (int d = threadIdx.x; d < D; d += 256) {
    float acc = 0.f;
    for (int c = 0; c < C; ++c) acc += p.cW[(size_t)c * D + d] * dy[c];
    dz[d] = acc;
    part += acc * zs[d];
  }
  sm[threadIdx.x] = part;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) sm[threadIdx.x] += sm[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) scal[3] = sm[0];
}

int pool_blocks(long long N) {
  long long g = (N + 15) / 16;
  if (g > 1024) g = 1024;
  if (g < 1) g = 1;
  return (int)g;
}

hipError_t launch_pool_fwd(const PoolArgs& p0, hipStream_t s) {
  PoolArgs p = p0;
  hipError_t e;
  if (p.use_mfma && pool_mfma_ok(p)) {
    // persistent grid: one workgroup per compute unit (the register-resident kernel fills it; the launchers of the others change the number)
    static int cus = 0;
    if (!cus) {
      int dev = 0;
      hipDeviceProp_t prop;
      if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
      if ((e = hipGetDeviceProperties(&prop, dev)) != hipSuccess) return e;
      cus = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 1;
    }
    long long groups = (p.N + 31) / 32;
    p.blocks = (int)(groups < cus ? groups : cus);
    if (p.blocks > 1024) p.blocks = 1024;
    e = launch_pool_gate_part_mfma(p, s);
  } else {
    e = launch_pool_gate_part_f32(p, s);
  }
  if (e != hipSuccess) return e;
  if (p.blocks > 1024) return hipErrorInvalidValue;
  const int nz = (p.D + 15) / 16;
  const long long na = p.alpha ? (p.N + 1023) / 1024 : 0;
  hipLaunchKernelGGL(pool_combine_k, dim3((unsigned)(nz + na)), dim3(256), 0, s, p, nz);
  return hipGetLastError();
}

}  // namespace sl
