// Bandwidth-bound element kernels: AbsMax INT8 activation quantiser (Sec. 3.1), weight statistics
// mu/lambda and the sign binariser/packer (Sec. 3.1, App. A), the router (Sec. 3.3).
#include <mutex>
#include <string.h>
#include "pq_internal.h"
#include "pq_pack.h"

// ------------------------------------------------------------------------------------------
// Activation quantiser: one wavefront per token.  The row is read once from HBM into registers
// (16 B per lane per step), the wave reduces |x| with cross-lane shuffles, then each lane
// quantises what it holds.  Rows too long for the register cache are re-read (second read hits L2).
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ int quant_code(float x, float g) {
  float y = __fmul_rn(x, g);                       // one fp32 product, no contraction
  float r = rintf(y);                              // round half to even
  r = fminf(fmaxf(r, -128.0f), 127.0f);
  return (int)r;
}

template <typename T, bool NT = false>
__device__ __forceinline__ void quant_store(const uint4& u, float g, int8_t* qrow, uint16_t* xtrow,
                                            int c) {
  constexpr int V = vec16<T>::V;
  float f[V];
  vec16<T>::unpack(u, f);
  int q[V];
#pragma unroll
  for (int j = 0; j < V; ++j) q[j] = quant_code(f[j], g);
  uint32_t w[V / 4];
#pragma unroll
  for (int j = 0; j < V / 4; ++j)
    w[j] = (uint32_t)(q[4 * j] & 0xFF) | ((uint32_t)(q[4 * j + 1] & 0xFF) << 8) |
           ((uint32_t)(q[4 * j + 2] & 0xFF) << 16) | ((uint32_t)(q[4 * j + 3] & 0xFF) << 24);
  if constexpr (V == 8) {
    pq_st8<NT>(qrow + (size_t)c * 8, make_uint2(w[0], w[1]));
  } else {
    *reinterpret_cast<uint32_t*>(qrow + (size_t)c * 4) = w[0];
  }
  if (xtrow) {
    uint32_t o[V / 2];
#pragma unroll
    for (int j = 0; j < V / 2; ++j)
      o[j] = pack_bf16x2((float)q[2 * j] / g, (float)q[2 * j + 1] / g);
    if constexpr (V == 8) {
      pq_st16<NT>(xtrow + (size_t)c * 8, make_uint4(o[0], o[1], o[2], o[3]));
    } else {
      pq_st8<NT>(xtrow + (size_t)c * 4, make_uint2(o[0], o[1]));
    }
  }
}

// one wavefront: the K elements at x become row `row` of the results
template <typename T, int NV>
__device__ __forceinline__ void quant_act_row(const T* __restrict__ x, int row, int K, int8_t* __restrict__ Xq,
                                              float* __restrict__ gamma, uint16_t* __restrict__ Xt) {
  constexpr int V = vec16<T>::V;
  const int lane = threadIdx.x & 63;
  const uint4* xr = reinterpret_cast<const uint4*>(x);
  const int nvec = K / V;
  float amax = 0.0f;
  uint4 cache[NV > 0 ? NV : 1];
  if constexpr (NV > 0) {
    // unconditional loads (lanes past the end re-read the last vector, which cannot change the maximum): a load
    // under a branch gets a wait of its own and the row would arrive one memory latency per vector
#pragma unroll
    for (int i = 0; i < NV; ++i) cache[i] = xr[min(i * 64 + lane, nvec - 1)];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      float f[V];
      vec16<T>::unpack(cache[i], f);
#pragma unroll
      for (int j = 0; j < V; ++j) amax = fmaxf(amax, fabsf(f[j]));
    }
  } else {
    for (int c = lane; c < nvec; c += 64) {
      uint4 u = xr[c];
      float f[V];
      vec16<T>::unpack(u, f);
#pragma unroll
      for (int j = 0; j < V; ++j) amax = fmaxf(amax, fabsf(f[j]));
    }
  }
  amax = wave_max(amax);
  const float g = 128.0f / fmaxf(amax, 1e-5f);     // IEEE fp32 division (no fast-math in this build)
  if (lane == 0) gamma[row] = g;
  int8_t* qrow = Xq + (size_t)row * K;
  uint16_t* xtrow = Xt ? Xt + (size_t)row * K : nullptr;
  if constexpr (NV > 0) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      int c = i * 64 + lane;
      if (c < nvec) quant_store<T>(cache[i], g, qrow, xtrow, c);
    }
  } else {
    for (int c = lane; c < nvec; c += 64) quant_store<T>(xr[c], g, qrow, xtrow, c);
  }
}

template <typename T, int NV>
__device__ __forceinline__ void quant_act_body(const T* __restrict__ X, int Tn, int K, int8_t* __restrict__ Xq,
                                               float* __restrict__ gamma, uint16_t* __restrict__ Xt, int block) {
  const int row = block * 4 + (threadIdx.x >> 6);
  if (row < Tn) quant_act_row<T, NV>(X + (size_t)row * K, row, K, Xq, gamma, Xt);
}

template <typename T, int NV>
__global__ __launch_bounds__(256) void quant_act_kernel(const T* __restrict__ X, int Tn, int K,
                                                        int8_t* __restrict__ Xq,
                                                        float* __restrict__ gamma,
                                                        uint16_t* __restrict__ Xt) {
  quant_act_body<T, NV>(X, Tn, K, Xq, gamma, Xt, blockIdx.x);
}

// The gated unit of INT8 experts and the quantiser of its result: a = bf16(silu(g) u) over rows of r elements (u and g of a row ld
// elements apart from the next row's), then what quant_act_row makes of a.  Bound by its launch at most sizes; with a in memory
// between two launches the FFN of 2048 tokens 2048/5076, r = 384 took 607.9 us, so 604.9.  Rows of up to 64 NV vectors stay in registers.
template <int NV>
__global__ __launch_bounds__(256) void expert_act_quant_kernel(const uint16_t* __restrict__ ue, const uint16_t* __restrict__ ge, int ld, int S,
                                                               int r, int8_t* __restrict__ aq, float* __restrict__ gamma,
                                                               uint16_t* __restrict__ at) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= S) return;
  const uint4* u4 = reinterpret_cast<const uint4*>(ue + (size_t)row * ld);
  const uint4* g4 = reinterpret_cast<const uint4*>(ge + (size_t)row * ld);
  const int nvec = r / 8;
  uint4 uv[NV], gv[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = min(i * 64 + lane, nvec - 1);      // (past the end: the last vector again, which cannot change the maximum)
    uv[i] = u4[c];
    gv[i] = g4[c];
  }
  float amax = 0.0f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    float u[8], g[8];
    vec16<uint16_t>::unpack(uv[i], u);
    vec16<uint16_t>::unpack(gv[i], g);
#pragma unroll
    for (int j = 0; j < 8; ++j) u[j] = pq_silu(g[j]) * u[j];
    uv[i] = make_uint4(pack_bf16x2(u[0], u[1]), pack_bf16x2(u[2], u[3]), pack_bf16x2(u[4], u[5]), pack_bf16x2(u[6], u[7]));
    vec16<uint16_t>::unpack(uv[i], u);
#pragma unroll
    for (int j = 0; j < 8; ++j) amax = fmaxf(amax, fabsf(u[j]));
  }
  amax = wave_max(amax);
  const float g = 128.0f / fmaxf(amax, 1e-5f);
  if (lane == 0) gamma[row] = g;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = i * 64 + lane;
    if (c < nvec) quant_store<uint16_t>(uv[i], g, aq + (size_t)row * r, at + (size_t)row * r, c);
  }
}

bool pq_expert_act_quant_applies(int r) { return r <= 2048; }
int pq_launch_expert_act_quant(const void* ue, const void* ge, int ld, int S, int r, int8_t* aq, float* gamma, void* at, hipStream_t s) {
  if (S == 0) return PQ_OK;
  pq_prof_scope prof(PQP_MOE_ELEMENTWISE, s);
  const dim3 grid((S + 3) / 4), block(256);
  const uint16_t *u = (const uint16_t*)ue, *g = (const uint16_t*)ge;
  if (r <= 512) expert_act_quant_kernel<1><<<grid, block, 0, s>>>(u, g, ld, S, r, aq, gamma, (uint16_t*)at);
  else if (r <= 2048) expert_act_quant_kernel<4><<<grid, block, 0, s>>>(u, g, ld, S, r, aq, gamma, (uint16_t*)at);
  else return pq_set_error(PQ_ERR_SHAPE, "rows of %d elements do not fit the registers of the expert quantiser", r);
  PQ_CHECK_LAUNCH("expert_act_quant_kernel");
  return PQ_OK;
}

template <typename T>
static int launch_quant_t(const T* X, int Tn, int K, int8_t* Xq, float* gamma, uint16_t* Xt,
                          hipStream_t s) {
  constexpr int V = vec16<T>::V;
  const int per_lane = (K / V + 63) / 64;
  dim3 grid((Tn + 3) / 4), block(256);
  if (per_lane <= 4) quant_act_kernel<T, 4><<<grid, block, 0, s>>>(X, Tn, K, Xq, gamma, Xt);
  else if (per_lane <= 8) quant_act_kernel<T, 8><<<grid, block, 0, s>>>(X, Tn, K, Xq, gamma, Xt);
  else if (per_lane <= 16) quant_act_kernel<T, 16><<<grid, block, 0, s>>>(X, Tn, K, Xq, gamma, Xt);
  else quant_act_kernel<T, 0><<<grid, block, 0, s>>>(X, Tn, K, Xq, gamma, Xt);
  PQ_CHECK_LAUNCH("quant_act_kernel");
  return PQ_OK;
}

int pq_launch_quant_act(const void* X, int dtype, int T, int K, int8_t* Xq, float* gamma,
                        uint16_t* Xt, hipStream_t s) {
  if (T == 0) return PQ_OK;
  pq_prof_scope prof(PQP_QUANT, s);
  if (dtype == PQ_F32) return launch_quant_t<float>((const float*)X, T, K, Xq, gamma, Xt, s);
  return launch_quant_t<uint16_t>((const uint16_t*)X, T, K, Xq, gamma, Xt, s);
}

// ------------------------------------------------------------------------------------------
// Weight statistics, stage 1: grid-stride fp64 sums of W and |W|, one pair per block.
// ------------------------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ void wstats_partial_body(const T* __restrict__ W, size_t nvec, double* __restrict__ partials, int block,
                                                    int nblocks) {
  constexpr int V = vec16<T>::V;
  __shared__ double red[4];
  const uint4* w4 = reinterpret_cast<const uint4*>(W);
  double s = 0.0, a = 0.0;
  for (size_t c = (size_t)block * 256 + threadIdx.x; c < nvec; c += (size_t)nblocks * 256) {
    float f[V];
    vec16<T>::unpack(w4[c], f);
#pragma unroll
    for (int j = 0; j < V; ++j) {
      s += (double)f[j];
      a += (double)fabsf(f[j]);
    }
  }
  double bs = block_sum_d<256>(s, red);
  double ba = block_sum_d<256>(a, red);
  if (threadIdx.x == 0) {
    partials[2 * block] = bs;
    partials[2 * block + 1] = ba;
  }
}

// ------------------------------------------------------------------------------------------
// RMSNorm fused with the AbsMax quantiser (Sec. 3.1: Q(Norm(X)); App. A: both are element-wise per token
// and merge; App. B: RMSNorm).  One wavefront per token, the row stays in registers between the three
// steps: sum of squares (fp64, so that rstd does not depend on the order of the sum beyond its last fp64
// bit), x_hat = fl(fl(x rstd) g) rounded to the I/O type, then the quantiser of the stored x_hat.  The first nw workgroups
// take the first stage of a weight's statistics instead (a linear with its normalisation: as a launch of their own they
// were 5 us of the 230 of forward and backward of 4096 tokens 2048x2048, within this one 1).
// ------------------------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ uint4 pack_io(const float* f);
template <>
__device__ __forceinline__ uint4 pack_io<float>(const float* f) {
  return make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3]));
}
template <>
__device__ __forceinline__ uint4 pack_io<uint16_t>(const float* f) {
  return make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7]));
}

template <typename T, int NV>
__global__ __launch_bounds__(256) void rmsnorm_quant_kernel(const T* __restrict__ X, const T* __restrict__ gain, int Tn, int K,
                                                            float eps, T* __restrict__ Xn, int8_t* __restrict__ Xq,
                                                            float* __restrict__ gamma, uint16_t* __restrict__ Xt,
                                                            float* __restrict__ rstd_out, const T* __restrict__ W, size_t w_vecs,
                                                            double* __restrict__ partials, int nw) {
  if ((int)blockIdx.x < nw) {                        // uniform
    wstats_partial_body<T>(W, w_vecs, partials, blockIdx.x, nw);
    return;
  }
  constexpr int V = vec16<T>::V;
  const int lane = threadIdx.x & 63;
  const int row = (blockIdx.x - nw) * 4 + (threadIdx.x >> 6);
  if (row >= Tn) return;
  const uint4* xr = reinterpret_cast<const uint4*>(X + (size_t)row * K);
  const uint4* gr = reinterpret_cast<const uint4*>(gain);
  const int nvec = K / V;
  uint4 cache[NV], gc[NV];
  double ss = 0.0;
  // unconditional loads (clamped index) so that all of them are in flight together
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int cc = min(i * 64 + lane, nvec - 1);
    cache[i] = xr[cc];
    gc[i] = gr[cc];
  }
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    if (i * 64 + lane < nvec) {
      float f[V];
      vec16<T>::unpack(cache[i], f);
#pragma unroll
      for (int j = 0; j < V; ++j) ss += (double)f[j] * (double)f[j];
    }
  }
  ss = wave_sum_d(ss);
  const float r = (float)(1.0 / sqrt(ss / (double)K + (double)eps));
  float amax = 0.0f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = i * 64 + lane;
    if (c < nvec) {
      float f[V], g[V];
      vec16<T>::unpack(cache[i], f);
      vec16<T>::unpack(gc[i], g);
#pragma unroll
      for (int j = 0; j < V; ++j) f[j] = __fmul_rn(__fmul_rn(f[j], r), g[j]);
      cache[i] = pack_io<T>(f);                      // the stored x_hat; everything below reads it back
      vec16<T>::unpack(cache[i], f);
#pragma unroll
      for (int j = 0; j < V; ++j) amax = fmaxf(amax, fabsf(f[j]));
      if (Xn) pq_st16<true>(reinterpret_cast<uint4*>(Xn + (size_t)row * K) + c, cache[i]);
    }
  }
  amax = wave_max(amax);
  const float g = 128.0f / fmaxf(amax, 1e-5f);
  if (lane == 0) {
    gamma[row] = g;
    if (rstd_out) rstd_out[row] = r;
  }
  int8_t* qrow = Xq + (size_t)row * K;
  uint16_t* xtrow = Xt ? Xt + (size_t)row * K : nullptr;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = i * 64 + lane;
    if (c < nvec) quant_store<T, true>(cache[i], g, qrow, xtrow, c);
  }
}

template <typename T>
static int launch_rmsnorm_quant_t(const T* X, const T* gain, int Tn, int K, float eps, T* Xn, int8_t* Xq, float* gamma,
                                  uint16_t* Xt, float* rstd, hipStream_t s, const T* W, size_t w_elems, double* partials, int nw) {
  constexpr int V = vec16<T>::V;
  const int per_lane = (K / V + 63) / 64;
  dim3 grid((Tn + 3) / 4 + nw), block(256);
  const size_t wv = w_elems / V;
  if (per_lane <= 4) rmsnorm_quant_kernel<T, 4><<<grid, block, 0, s>>>(X, gain, Tn, K, eps, Xn, Xq, gamma, Xt, rstd, W, wv, partials, nw);
  else if (per_lane <= 8) rmsnorm_quant_kernel<T, 8><<<grid, block, 0, s>>>(X, gain, Tn, K, eps, Xn, Xq, gamma, Xt, rstd, W, wv, partials, nw);
  else if (per_lane <= 16) rmsnorm_quant_kernel<T, 16><<<grid, block, 0, s>>>(X, gain, Tn, K, eps, Xn, Xq, gamma, Xt, rstd, W, wv, partials, nw);
  else return pq_set_error(PQ_ERR_SHAPE, "row of %d elements does not fit the register cache of the fused normalising quantiser", K);
  PQ_CHECK_LAUNCH("rmsnorm_quant_kernel");
  return PQ_OK;
}

int pq_launch_rmsnorm_quant(const void* X, const void* gain, int dtype, int T, int K, float eps, void* Xn, int8_t* Xq,
                            float* gamma, uint16_t* Xt, float* rstd, hipStream_t s, const void* W, size_t w_elems, double* partials, int nw) {
  if (T == 0 && nw == 0) return PQ_OK;
  pq_prof_scope prof(PQP_NORM_QUANT, s);
  if (dtype == PQ_F32)
    return launch_rmsnorm_quant_t<float>((const float*)X, (const float*)gain, T, K, eps, (float*)Xn, Xq, gamma, Xt, rstd, s, (const float*)W, w_elems, partials, nw);
  return launch_rmsnorm_quant_t<uint16_t>((const uint16_t*)X, (const uint16_t*)gain, T, K, eps, (uint16_t*)Xn, Xq, gamma, Xt, rstd, s, (const uint16_t*)W,
                                          w_elems, partials, nw);
}

// Backward of the normalisation (the quantiser is passed straight through, App. B.1): with u = x rstd,
//   dx = rstd (g dxn - u mean_k(g dxn u)),   dg[k] = sum_t dxn[t][k] u[t][k].
// A wavefront walks NORM_BWD_TPW tokens and keeps its share of dg in registers; the four wavefronts of a
// workgroup add their shares through LDS into one partial row, and a second kernel adds the partial rows in a
// fixed order (fp64), so the result is the same on every run.
constexpr int NORM_BWD_TPW = 4;                    // tokens per wavefront
constexpr int NORM_BWD_TPB = 4 * NORM_BWD_TPW;     // tokens per workgroup = per partial row of dgain

template <typename T, int NV>
__global__ __launch_bounds__(256) void rmsnorm_bwd_kernel(const T* __restrict__ dXn, const T* __restrict__ X,
                                                          const T* __restrict__ gain, const float* __restrict__ rstd, int Tn,
                                                          int K, T* __restrict__ dX, float* __restrict__ part) {
  constexpr int V = vec16<T>::V;
  extern __shared__ __attribute__((aligned(16))) float dsh[];   // [3][K]: the dgain shares of wavefronts 1..3
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t0 = blockIdx.x * NORM_BWD_TPB + wave * NORM_BWD_TPW;
  const int nvec = K / V;
  const uint4* gr = reinterpret_cast<const uint4*>(gain);
  uint4 gp[NV];
  float dga[NV][V];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    gp[i] = gr[min(i * 64 + lane, nvec - 1)];
#pragma unroll
    for (int j = 0; j < V; ++j) dga[i][j] = 0.0f;
  }
  const int t1 = min(t0 + NORM_BWD_TPW, Tn);
  for (int t = t0; t < t1; t += 2) {                  // two tokens per pass: sixteen row loads in flight
    const bool two = t + 1 < t1;
    const int tb = two ? t + 1 : t;
    uint4 dc[2][NV], xc[2][NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c = min(i * 64 + lane, nvec - 1);
      dc[0][i] = reinterpret_cast<const uint4*>(dXn + (size_t)t * K)[c];
      xc[0][i] = reinterpret_cast<const uint4*>(X + (size_t)t * K)[c];
      dc[1][i] = reinterpret_cast<const uint4*>(dXn + (size_t)tb * K)[c];
      xc[1][i] = reinterpret_cast<const uint4*>(X + (size_t)tb * K)[c];
    }
    const float s2[2] = {rstd[t], rstd[tb]};
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (q == 1 && !two) break;
      const float s = s2[q];
      double dot = 0.0;
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        if (i * 64 + lane < nvec) {
          float d[V], x[V], g[V];
          vec16<T>::unpack(dc[q][i], d);
          vec16<T>::unpack(xc[q][i], x);
          vec16<T>::unpack(gp[i], g);
#pragma unroll
          for (int j = 0; j < V; ++j) {
            const float u = __fmul_rn(x[j], s);
            dot += (double)__fmul_rn(g[j], d[j]) * (double)u;
            dga[i][j] = __fadd_rn(dga[i][j], __fmul_rn(d[j], u));
          }
        }
      }
      const float cm = (float)(wave_sum_d(dot) / (double)K);
      T* orow = dX + (size_t)(q ? tb : t) * K;
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int c = i * 64 + lane;
        if (c < nvec) {
          float d[V], x[V], g[V], o[V];
          vec16<T>::unpack(dc[q][i], d);
          vec16<T>::unpack(xc[q][i], x);
          vec16<T>::unpack(gp[i], g);
#pragma unroll
          for (int j = 0; j < V; ++j) {
            const float u = __fmul_rn(x[j], s);
            o[j] = __fmul_rn(s, __fsub_rn(__fmul_rn(g[j], d[j]), __fmul_rn(u, cm)));
          }
          pq_st16<true>(reinterpret_cast<uint4*>(orow) + c, pack_io<T>(o));
        }
      }
    }
  }
  // the four wavefronts' shares are added in wavefront order and leave as one partial row
  if (wave > 0) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c = i * 64 + lane;
      if (c < nvec) {
#pragma unroll
        for (int j = 0; j < V; j += 4)
          *reinterpret_cast<float4*>(dsh + (size_t)(wave - 1) * K + (size_t)c * V + j) =
              make_float4(dga[i][j], dga[i][j + 1], dga[i][j + 2], dga[i][j + 3]);
      }
    }
  }
  __syncthreads();
  if (wave == 0) {
    float* prow = part + (size_t)blockIdx.x * K;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c = i * 64 + lane;
      if (c < nvec) {
#pragma unroll
        for (int j = 0; j < V; j += 4) {
          float4 a = make_float4(dga[i][j], dga[i][j + 1], dga[i][j + 2], dga[i][j + 3]);
#pragma unroll
          for (int w = 0; w < 3; ++w) {
            const float4 b = *reinterpret_cast<const float4*>(dsh + (size_t)w * K + (size_t)c * V + j);
            a.x = __fadd_rn(a.x, b.x); a.y = __fadd_rn(a.y, b.y); a.z = __fadd_rn(a.z, b.z); a.w = __fadd_rn(a.w, b.w);
          }
          *reinterpret_cast<float4*>(prow + (size_t)c * V + j) = a;
        }
      }
    }
  }
}

// 8 columns x 32 row slices per workgroup: slice r adds rows r, r + 32, ... (sixteen independent loads in
// flight), the slices are then added in slice order.
__global__ __launch_bounds__(256) void rmsnorm_dgain_kernel(const float* __restrict__ part, int nrows, int K, float* __restrict__ dgain) {
  __shared__ double red[32][9];
  const int col = threadIdx.x & 7, slice = threadIdx.x >> 3;
  const int k = blockIdx.x * 8 + col;
  double a = 0.0;
  if (k < K) {
    int w = slice;
    for (; w + 15 * 32 < nrows; w += 16 * 32) {
      float v[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = part[(size_t)(w + 32 * i) * K + k];
#pragma unroll
      for (int i = 0; i < 16; ++i) a += (double)v[i];
    }
    for (; w < nrows; w += 32) a += (double)part[(size_t)w * K + k];
  }
  red[slice][col] = a;
  __syncthreads();
  if (slice == 0 && k < K) {
    double t = 0.0;
#pragma unroll
    for (int r = 0; r < 32; ++r) t += red[r][col];
    dgain[k] = (float)t;
  }
}

size_t pq_rmsnorm_bwd_scratch_bytes(int T, int K) {
  return (size_t)((T + NORM_BWD_TPB - 1) / NORM_BWD_TPB) * K * sizeof(float);
}

template <typename T>
static int launch_rmsnorm_bwd_t(const T* dXn, const T* X, const T* gain, const float* rstd, int Tn, int K, T* dX, float* part,
                                hipStream_t s) {
  constexpr int V = vec16<T>::V;
  const int per_lane = (K / V + 63) / 64;
  dim3 grid((Tn + NORM_BWD_TPB - 1) / NORM_BWD_TPB), block(256);
  const size_t lds = (size_t)3 * K * sizeof(float);
  if (per_lane <= 4) rmsnorm_bwd_kernel<T, 4><<<grid, block, lds, s>>>(dXn, X, gain, rstd, Tn, K, dX, part);
  else if (per_lane <= 8) rmsnorm_bwd_kernel<T, 8><<<grid, block, lds, s>>>(dXn, X, gain, rstd, Tn, K, dX, part);
  else return pq_set_error(PQ_ERR_SHAPE, "row of %d elements does not fit the register cache of the normalisation backward", K);
  PQ_CHECK_LAUNCH("rmsnorm_bwd_kernel");
  return PQ_OK;
}

int pq_launch_rmsnorm_bwd(const void* dXn, const void* X, const void* gain, const float* rstd, int dtype, int T, int K, void* dX,
                          float* dgain, float* part, hipStream_t s) {
  if (T > 0) {
    pq_prof_scope prof(PQP_NORM_BWD, s);
    int e;
    if (dtype == PQ_F32)
      e = launch_rmsnorm_bwd_t<float>((const float*)dXn, (const float*)X, (const float*)gain, rstd, T, K, (float*)dX, part, s);
    else
      e = launch_rmsnorm_bwd_t<uint16_t>((const uint16_t*)dXn, (const uint16_t*)X, (const uint16_t*)gain, rstd, T, K, (uint16_t*)dX, part, s);
    if (e) return e;
  }
  pq_prof_scope prof(PQP_NORM_BWD, s);
  rmsnorm_dgain_kernel<<<(K + 7) / 8, 256, 0, s>>>(part, (T + NORM_BWD_TPB - 1) / NORM_BWD_TPB, K, dgain);
  PQ_CHECK_LAUNCH("rmsnorm_dgain_kernel");
  return PQ_OK;
}

// ------------------------------------------------------------------------------------------
// Scratch for callers that cannot allocate (code under graph capture, serving loops): a file-scope device array
// that every GPU the library runs on holds until the process ends.  Its name is a host-side stand-in, not a
// device address: the address is looked up once per device and only that pointer is handed to kernels.
// ------------------------------------------------------------------------------------------
constexpr size_t PQ_STATIC_SCRATCH_BYTES = (size_t)4 << 20;
constexpr int PQ_MAX_DEVICES = 64;
static __device__ __align__(256) unsigned char scratch[PQ_STATIC_SCRATCH_BYTES];
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[PQ_MAX_DEVICES];

size_t pq_static_scratch_bytes() { return PQ_STATIC_SCRATCH_BYTES; }

int pq_static_scratch(void** out) {
  int dev = -1;
  PQ_CHECK_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= PQ_MAX_DEVICES) return pq_set_error(PQ_ERR_HIP, "device ordinal %d is outside 0..%d", dev, PQ_MAX_DEVICES - 1);
  std::lock_guard<std::mutex> g(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    PQ_CHECK_HIP(hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return pq_set_error(PQ_ERR_HIP, "hipGetSymbolAddress returned a NULL address for the static scratch");
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return PQ_OK;
}

template <typename T>
__global__ __launch_bounds__(256) void wstats_partial_kernel(const T* __restrict__ W, size_t nvec,
                                                             double* __restrict__ partials) {
  wstats_partial_body<T>(W, nvec, partials, blockIdx.x, gridDim.x);
}

// ------------------------------------------------------------------------------------------
// Router: a wavefront takes TB tokens at once (a router row converted to fp64 serves all of them): fp64 dot products
// against all E router rows, lane l accumulating the 16-byte chunks l, l + 64, ... of a token row in order, then the
// wave sums, which leave one (token, expert) pair per lane; that lane rounds the logit to fp32 and evaluates its term
// of the softmax in fp64; the first lane of a token's group selects the top-k (ties to the lower index).
// ------------------------------------------------------------------------------------------
// hist (may be NULL): [workgroups][E], how many slots of the workgroup's 4 TB tokens each expert got (what the permutation starts from).
template <typename T, int EMAX, int TB>
__device__ __forceinline__ void router_body(const T* __restrict__ X, const T* __restrict__ Wr, int Tn, int K, int E, int k, int* __restrict__ idx,
                                            float* __restrict__ gate, float* __restrict__ probs, int* __restrict__ hist, int block) {
  constexpr int V = vec16<T>::V;
  __shared__ int s_hist[64];
  const int lane = threadIdx.x & 63;
  const int t0 = (block * 4 + (threadIdx.x >> 6)) * TB;
  if (hist) {                                        // uniform
    if (threadIdx.x < 64) s_hist[threadIdx.x] = 0;
    __syncthreads();
  } else if (t0 >= Tn) return;
  const int nvec = K / V;
  double acc[TB][EMAX];
#pragma unroll
  for (int tb = 0; tb < TB; ++tb)
#pragma unroll
    for (int e = 0; e < EMAX; ++e) acc[tb][e] = 0.0;
  // Router rows are requested unconditionally, eight at a time (rows past E repeat the last one and their sums
  // are never used; tokens past the end repeat the last token): a load under a branch gets a wait of its own, which
  // made this loop a chain of latencies.
  for (int c = lane; c < nvec; c += 64) {
    double xd[TB][V];
    uint4 xv[TB];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) xv[tb] = reinterpret_cast<const uint4*>(X + (size_t)min(t0 + tb, Tn - 1) * K)[c];
#pragma unroll
    for (int e0 = 0; e0 < EMAX; e0 += 8) {
      uint4 wv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) wv[u] = reinterpret_cast<const uint4*>(Wr + (size_t)min(e0 + u, E - 1) * K)[c];
      if (e0 == 0) {
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
          float xf[V];
          vec16<T>::unpack(xv[tb], xf);
#pragma unroll
          for (int j = 0; j < V; ++j) xd[tb][j] = (double)xf[j];
        }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        float wf[V];
        vec16<T>::unpack(wv[u], wf);
#pragma unroll
        for (int j = 0; j < V; ++j) {
          const double wd = (double)wf[j];
#pragma unroll
          for (int tb = 0; tb < TB; ++tb) acc[tb][e0 + u] += xd[tb][j] * wd;
        }
      }
    }
  }
  // Sums over the wavefront, transposed (see wave_sum_transposed): lane l ends with the sum of value l / ST.
  constexpr int NV = TB * EMAX, ST = 64 / NV;
  static_assert(NV == 32 || NV == 64, "a wavefront carries 32 or 64 (token, expert) sums");
  double v[NV];
#pragma unroll
  for (int tb = 0; tb < TB; ++tb)
#pragma unroll
    for (int e = 0; e < EMAX; ++e) v[tb * EMAX + e] = acc[tb][e];
  wave_sum_transposed<NV, 32>(v, lane);
  // lane l: pair (token tb, expert e); one exponential and one division per lane
  const int vi = lane / ST, tb = vi / EMAX, e = vi % EMAX;
  const double lg = (double)(float)v[0];              // one rounding to fp32
  const bool live = e < E;
  double mx = live ? lg : -1e300;
#pragma unroll
  for (int off = ST; off < ST * EMAX; off <<= 1) mx = fmax(mx, __shfl_xor(mx, off, 64));
  double pr = live ? exp(lg - mx) : 0.0;
  double den = pr;
#pragma unroll
  for (int off = ST; off < ST * EMAX; off <<= 1) den += __shfl_xor(den, off, 64);
  pr /= den;
  const int t = t0 + tb;
  if (probs && live && t < Tn && lane % ST == 0) probs[(size_t)t * E + e] = (float)pr;
  // the token's logits and probabilities into every lane of its group, then the top-k (ties to the lower index)
  double logit[EMAX], p[EMAX];
#pragma unroll
  for (int ee = 0; ee < EMAX; ++ee) {
    logit[ee] = __shfl(lg, (tb * EMAX + ee) * ST, 64);
    p[ee] = __shfl(pr, (tb * EMAX + ee) * ST, 64);
  }
  if (lane % (ST * EMAX) == 0 && t < Tn) {            // the group's first lane writes the token's choice
    unsigned long long taken = 0ull;
    for (int j = 0; j < k; ++j) {
      int best = -1;
      double bv = 0.0, bp = 0.0;
#pragma unroll
      for (int ee = 0; ee < EMAX; ++ee) {
        if (ee < E && !((taken >> ee) & 1ull) && (best < 0 || logit[ee] > bv)) {
          best = ee; bv = logit[ee]; bp = p[ee];
        }
      }
      taken |= 1ull << best;
      idx[(size_t)t * k + j] = best;
      gate[(size_t)t * k + j] = (float)bp;
      if (hist) atomicAdd(&s_hist[best], 1);
    }
  }
  if (hist) {
    __syncthreads();
    if ((int)threadIdx.x < E) hist[(size_t)block * E + threadIdx.x] = s_hist[threadIdx.x];
  }
}
template <typename T, int EMAX, int TB>
__global__ __launch_bounds__(256) void router_kernel(const T* __restrict__ X, const T* __restrict__ Wr, int Tn, int K, int E, int k,
                                                     int* __restrict__ idx, float* __restrict__ gate, float* __restrict__ probs, int* __restrict__ hist) {
  router_body<T, EMAX, TB>(X, Wr, Tn, K, E, k, idx, gate, probs, hist, blockIdx.x);
}
// tokens of a router workgroup
int pq_router_tokens(int E) { return E <= 8 ? 16 : E <= 16 ? 8 : 4; }


// ------------------------------------------------------------------------------------------
// The slots (slot = token * k + j) ordered by expert, slots of one expert in their own order: perm[pos] = slot, inv[slot] = pos,
// offsets[e] = first position of expert e, and with it the slots' rows of the activations, copied to dst[pos].
// The router's workgroups have counted their experts (hist).  A workgroup here owns a run of them: it sums what lies before it and in
// all, per expert, which gives it the first position of each expert's slots, walks its own slots 64 at a time (rank inside a batch by
// ballot prefix, lane e carrying expert e's running position) and copies their rows.  Any number of workgroups: as a counting sort on
// one workgroup and a gather in a launch of its own the two took 15 + 12 us for 8192 tokens, 25 + 22 for 16384 (2048 wide).  Every workgroup
// reads all counts: with 64 experts and 65536 tokens (two active, 512 wide) that is 349 us of the 3070 of a whole call, which the counting sort made 4044.
// ------------------------------------------------------------------------------------------
constexpr int PLACE_GROUPS = 512;                    // workgroups at most (each reads all of hist)
// sub of subs: while there are few runs each goes to several workgroups, which all find its positions and copy every subs-th row
__device__ __forceinline__ void place_body(const pq_place p, int wg, int groups, int subs) {
  const int g = wg / subs, sub = wg - g * subs;
  constexpr int SMAX = 256;                          // slots of a router workgroup: 16 tokens x 8, 8 x 16 or 4 x 64 experts
  __shared__ int s_pre[256], s_all[256], s_run[64], s_pos[SMAX];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, E = p.E;
  const int per = (p.nblk + groups - 1) / groups, b0 = min(g * per, p.nblk), b1 = min(b0 + per, p.nblk);
  {  // thread (e, j): expert e over every J-th workgroup of the router
    const int J = 256 / E, e = tid % E, j = tid / E;
    int pre = 0, all = 0;
    if (j < J) {
      for (int w0 = j; w0 < p.nblk; w0 += 8 * J) {   // (eight loads in flight, clamped)
        int v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p.hist[(size_t)min(w0 + u * J, p.nblk - 1) * E + e];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int w = w0 + u * J;
          all += w < p.nblk ? v[u] : 0;
          pre += w < b0 ? v[u] : 0;
        }
      }
    }
    s_pre[tid] = pre;
    s_all[tid] = all;
    __syncthreads();
    if (wave == 0) {                                 // lane e: expert e
      int before = 0, total = 0;
      if (lane < E)
        for (int q = 0; q < J; ++q) { before += s_pre[q * E + lane]; total += s_all[q * E + lane]; }
      int incl = total;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int up = __shfl_up(incl, d);
        if (lane >= d) incl += up;
      }
      s_run[lane] = incl - total + before;
      if (wg == 0) {
        if (lane < E) {
          p.offsets[lane] = incl - total;
          p.counts[lane] = total;
        }
        if (lane == E - 1) p.offsets[E] = incl;
      }
    }
    __syncthreads();
  }
  for (int b = b0; b < b1; ++b) {                    // uniform
    const int t0 = b * p.tokens, n = min(p.tokens, p.T - t0) * p.k, slot0 = t0 * p.k;
    if (wave == 0) {
      int running = s_run[lane];
      for (int s0 = 0; s0 < n; s0 += 64) {
        const int s = s0 + lane, id = s < n ? p.idx[slot0 + s] : -1;
        int pos = 0;
        for (int e = 0; e < E; ++e) {
          const unsigned long long m = __ballot(id == e);
          const int base = __builtin_amdgcn_readlane(running, e);   // (e is uniform)
          if (id == e) pos = base + __builtin_popcountll(m & ((1ull << lane) - 1ull));
          if (lane == e) running += __builtin_popcountll(m);
        }
        if (s < n) {
          s_pos[s] = pos;
          if (sub == 0) {
            p.perm[pos] = slot0 + s;
            p.inv[slot0 + s] = pos;
          }
        }
      }
      s_run[lane] = running;
    }
    __syncthreads();
    const int nv = p.d / 8;
    for (int i = wave * subs + sub; i < n; i += 4 * subs) {   // a wavefront copies a row, up to four vectors of a lane in flight
      const size_t t = (size_t)(t0 + i / p.k), pos = (size_t)s_pos[i];
      const uint4* src = reinterpret_cast<const uint4*>(p.src + t * p.d);
      uint4* dst = reinterpret_cast<uint4*>(p.dst + pos * p.d);
      for (int c0 = lane; c0 < nv; c0 += 256) {
        const uint4 v0 = src[c0], v1 = src[min(c0 + 64, nv - 1)], v2 = src[min(c0 + 128, nv - 1)], v3 = src[min(c0 + 192, nv - 1)];
        dst[c0] = v0;
        if (c0 + 64 < nv) dst[c0 + 64] = v1;
        if (c0 + 128 < nv) dst[c0 + 128] = v2;
        if (c0 + 192 < nv) dst[c0 + 192] = v3;
      }
      if (p.codes) {                                 // uniform: INT8 experts, the row's codes and gamma too (d % 16 == 0)
        const uint4* q = reinterpret_cast<const uint4*>(p.codes + t * p.d);
        uint4* qo = reinterpret_cast<uint4*>(p.codes_out + pos * p.d);
        for (int c = lane; c < p.d / 16; c += 64) qo[c] = q[c];
        if (lane == 0) p.gamma_out[pos] = p.gamma[t];
      }
    }
    __syncthreads();
  }
}
static int place_groups(int nblk) { return nblk < 1 ? 1 : nblk < PLACE_GROUPS ? nblk : PLACE_GROUPS; }
static int place_subs(int nblk) { return nblk <= PLACE_GROUPS / 4 ? 4 : nblk <= PLACE_GROUPS / 2 ? 2 : 1; }

// The first stage of the weight statistics and the activation quantiser of one forward call are independent and
// each too short to fill its own launch well: one launch, the first nw workgroups take the weights.
struct slab_sum_job { const float* part; int splits, M, N; uint16_t* C; int ldc; };
template <typename T, int NV>
__global__ __launch_bounds__(256) void wstats_quant_kernel(const T* __restrict__ W, size_t nvec, double* __restrict__ partials,
                                                           int nw, const T* __restrict__ X, int Tn, int K,
                                                           int8_t* __restrict__ Xq, float* __restrict__ gamma,
                                                           uint16_t* __restrict__ Xt, int nq, slab_sum_job sj) {
  const int b = blockIdx.x;
  if (b < nw) wstats_partial_body<T>(W, nvec, partials, b, nw);
  else if (b < nw + nq) quant_act_body<T, NV>(X, Tn, K, Xq, gamma, Xt, b - nw);
  else pq_slab_sum_bf16_body(sj.part, sj.splits, sj.M, sj.N, sj.C, sj.ldc, (size_t)(b - nw - nq) * 256 + threadIdx.x);
}

// ... and the router of a call with up to eight experts, which reads the same activations (its workgroups, bound by fp64 sums, first).
template <int NV>
__global__ __launch_bounds__(256) void wstats_quant_router_kernel(const uint16_t* __restrict__ W, size_t nvec, double* __restrict__ partials,
                                                                  int nw, const uint16_t* __restrict__ X, int Tn, int K, int8_t* __restrict__ Xq,
                                                                  float* __restrict__ gamma, uint16_t* __restrict__ Xt, pq_router_job r, int nr) {
  const int b = blockIdx.x;
  if (b < nr) router_body<uint16_t, 8, 4>(X, (const uint16_t*)r.Wr, Tn, K, r.E, r.k, r.idx, r.gate, r.probs, r.hist, b);
  else if (b < nr + nw) wstats_partial_body<uint16_t>(W, nvec, partials, b - nr, nw);
  else quant_act_body<uint16_t, NV>(X, Tn, K, Xq, gamma, Xt, b - nr - nw);
}
// The router's registers leave two wavefronts to a SIMD, which the quantiser feels where it is bound by memory rather than by its
// launch.  Forward and backward with the router in a launch of its own / with it here (us): routed linears 2048x2048 of 256 tokens
// (320 workgroups of statistics and rows) 126.7 / 121.7, 2048 tokens (768) 206.1 / 200.0, 8192 tokens (2304) 404.1 / 401.0; FFNs
// 2048/5504 of 1024 tokens (2320) 433.5 / 433.4, 4096 tokens (3088) 919.6 / 924.0.
bool pq_wstats_quant_router_applies(int E, int K, long blocks) { return E <= 8 && K <= 4096 && blocks <= 2304; }
int pq_launch_wstats_quant_router(const void* W, size_t n_elems, double* partials, int nblocks, const void* X, int T, int K, int8_t* Xq, float* gamma,
                                  uint16_t* Xt, const pq_router_job& r, hipStream_t s) {
  if (T <= 0 || r.E > 8 || K > 4096) return pq_set_error(PQ_ERR_SHAPE, "combined statistics/quantiser/router launch: T=%d K=%d E=%d", T, K, r.E);
  pq_prof_scope prof(PQP_QUANT, s);
  const int nr = (T + 15) / 16, grid = nr + nblocks + (T + 3) / 4;
  const uint16_t *w = (const uint16_t*)W, *x = (const uint16_t*)X;
  if (K <= 2048) wstats_quant_router_kernel<4><<<grid, 256, 0, s>>>(w, n_elems / 8, partials, nblocks, x, T, K, Xq, gamma, Xt, r, nr);
  else wstats_quant_router_kernel<8><<<grid, 256, 0, s>>>(w, n_elems / 8, partials, nblocks, x, T, K, Xq, gamma, Xt, r, nr);
  PQ_CHECK_LAUNCH("wstats_quant_router_kernel");
  return PQ_OK;
}

// The weight side of the FFN's forward ahead of the packing, and the quantiser of its activations, as one launch (bf16): the
// statistics of up to three weights, the rows of X, the expert rows [Up_e; Gate_e] of every expert as one matrix, copied or
// (INT8 experts) put on the AbsMax grid, and the rows of Down_e likewise.  All independent and short: one after the other
// they were up to seven launches of which each costs a launch of about 5 us whatever it does.  With the packing in one launch and
// U, G and dW_up, dW_gate paired: FFN step at 153 tokens 992/2136 244 -> 203 us, 3135 tokens 320/924 249 -> 201 us, 4284 tokens
// 1728/2336 716 -> 668 us, 2048 tokens 2048/5076 703 -> 678 us.
// ROUTE: with the router of up to eight experts, whose workgroups come first.
template <int NV, bool ROUTE>
__global__ __launch_bounds__(256) void ffn_prep_kernel(pq_ffn_prep p) {
  int b = blockIdx.x;
  if constexpr (ROUTE) {
    const int nr = (p.T + 15) / 16;
    if (b < nr) {                                    // uniform
      router_body<uint16_t, 8, 4>((const uint16_t*)p.X, (const uint16_t*)p.route.Wr, p.T, p.D, p.E, p.route.k, p.route.idx, p.route.gate, p.route.probs,
                                  p.route.hist, b);
      return;
    }
    b -= nr;
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    if (b < p.w[i].nblocks) {                        // uniform
      wstats_partial_body<uint16_t>((const uint16_t*)p.w[i].W, (size_t)p.w[i].N * p.w[i].K / 8, p.w[i].partials, b, p.w[i].nblocks);
      return;
    }
    b -= p.w[i].nblocks;
  }
  const int nq = (p.T + 3) / 4;
  if (b < nq) {
    quant_act_body<uint16_t, NV>((const uint16_t*)p.X, p.T, p.D, p.Xq, p.gamma, p.Xt, b);
    return;
  }
  b -= nq;
  const int nug = p.E * 2 * p.r;
  if (p.UGQ) {
    if (b < (nug + 3) / 4) {
      const int row = b * 4 + (threadIdx.x >> 6);
      if (row >= nug) return;
      const int e = row / (2 * p.r), j = row - e * 2 * p.r;
      const uint16_t* src = j < p.r ? (const uint16_t*)p.Up + ((size_t)e * p.r + j) * p.D : (const uint16_t*)p.Gate + ((size_t)e * p.r + j - p.r) * p.D;
      quant_act_row<uint16_t, NV>(src, row, p.D, p.UGQ, p.gUG, p.UGT);
      return;
    }
    b -= (nug + 3) / 4;
    quant_act_body<uint16_t, 0>((const uint16_t*)p.Down, p.E * p.D, p.r, p.DownQ, p.gDown, p.DownT, b);
    return;
  }
  const size_t c = (size_t)b * 256 + threadIdx.x;    // UG[e][j][:] = Up[e][j][:] for j < r, Gate[e][j - r][:] for r <= j < 2 r
  const size_t nd = p.D / 8;
  if (c >= (size_t)nug * nd) return;
  const size_t row = c / nd, ch = c - row * nd, e = row / (size_t)(2 * p.r), j = row - e * (size_t)(2 * p.r);
  const uint16_t* src = j < (size_t)p.r ? (const uint16_t*)p.Up + (e * p.r + j) * p.D : (const uint16_t*)p.Gate + (e * p.r + (j - p.r)) * p.D;
  reinterpret_cast<uint4*>(p.UG)[c] = reinterpret_cast<const uint4*>(src)[ch];
}

int pq_launch_ffn_prep(const pq_ffn_prep& p, hipStream_t s) {
  pq_prof_scope prof(PQP_QUANT, s);
  const int per_lane = (p.D / 8 + 63) / 64, nug = p.E * 2 * p.r;
  long blocks = (long)(p.T + 3) / 4;
  for (const pq_weight_job& w : p.w) blocks += w.nblocks;
  if (p.UGQ) blocks += (nug + 3) / 4 + ((long)p.E * p.D + 3) / 4;
  else blocks += ((long)nug * (p.D / 8) + 255) / 256;
  if (p.route.Wr) {
    if (p.E > 8 || p.D > 4096) return pq_set_error(PQ_ERR_SHAPE, "router of %d experts in the launch of the statistics", p.E);
    blocks += (p.T + 15) / 16;
    if (per_lane <= 4) ffn_prep_kernel<4, true><<<(unsigned)blocks, 256, 0, s>>>(p);
    else ffn_prep_kernel<8, true><<<(unsigned)blocks, 256, 0, s>>>(p);
  } else if (per_lane <= 4) ffn_prep_kernel<4, false><<<(unsigned)blocks, 256, 0, s>>>(p);
  else if (per_lane <= 8) ffn_prep_kernel<8, false><<<(unsigned)blocks, 256, 0, s>>>(p);
  else if (per_lane <= 16) ffn_prep_kernel<16, false><<<(unsigned)blocks, 256, 0, s>>>(p);
  else ffn_prep_kernel<0, false><<<(unsigned)blocks, 256, 0, s>>>(p);
  PQ_CHECK_LAUNCH("ffn_prep_kernel");
  return PQ_OK;
}

// rows too long for the register-cached quantiser (more than 16 vectors per lane) take two launches
template <typename T>
static int launch_wstats_quant_t(const T* w, size_t n_elems, double* partials, int nblocks, const T* x, int Tn, int K, int8_t* Xq,
                                 float* gamma, uint16_t* Xt, hipStream_t s, const slab_sum_job& sj) {
  constexpr int V = vec16<T>::V;
  const int per_lane = (K / V + 63) / 64;
  if (Tn <= 0 || per_lane > 16) return pq_set_error(PQ_ERR_SHAPE, "combined statistics/quantiser launch: bad shape T=%d K=%d", Tn, K);
  pq_prof_scope prof(PQP_QUANT, s);
  const int nq = (Tn + 3) / 4;
  const int ns = sj.part ? (int)(((size_t)sj.M * (sj.N / 8) + 255) / 256) : 0;
  dim3 grid(nblocks + nq + ns), block(256);
  const size_t nvec = n_elems / V;
  if (per_lane <= 4) wstats_quant_kernel<T, 4><<<grid, block, 0, s>>>(w, nvec, partials, nblocks, x, Tn, K, Xq, gamma, Xt, nq, sj);
  else if (per_lane <= 8) wstats_quant_kernel<T, 8><<<grid, block, 0, s>>>(w, nvec, partials, nblocks, x, Tn, K, Xq, gamma, Xt, nq, sj);
  else wstats_quant_kernel<T, 16><<<grid, block, 0, s>>>(w, nvec, partials, nblocks, x, Tn, K, Xq, gamma, Xt, nq, sj);
  PQ_CHECK_LAUNCH("wstats_quant_kernel");
  return PQ_OK;
}

int pq_launch_wstats_quant(const void* W, int dtype, size_t n_elems, double* partials, int nblocks, const void* X, int T, int K,
                           int8_t* Xq, float* gamma, uint16_t* Xt, hipStream_t s, const float* slabs, int splits, int M, int N,
                           void* C, int ldc) {
  const slab_sum_job sj{slabs, splits, M, N, (uint16_t*)C, ldc};
  if (dtype == PQ_F32)
    return launch_wstats_quant_t<float>((const float*)W, n_elems, partials, nblocks, (const float*)X, T, K, Xq, gamma, Xt, s, sj);
  return launch_wstats_quant_t<uint16_t>((const uint16_t*)W, n_elems, partials, nblocks, (const uint16_t*)X, T, K, Xq, gamma, Xt, s, sj);
}

int pq_stats_blocks(size_t n_elems) {
  size_t b = (n_elems / 8 + 256 * 8 - 1) / (256 * 8);
  if (b < 1) b = 1;
  if (b > 1024) b = 1024;
  return (int)b;
}

int pq_launch_wstats_partial(const void* W, int dtype, size_t n_elems, double* partials, int nblocks,
                             hipStream_t s) {
  pq_prof_scope prof(PQP_WSTATS, s);
  if (dtype == PQ_F32)
    wstats_partial_kernel<float><<<nblocks, 256, 0, s>>>((const float*)W, n_elems / 4, partials);
  else
    wstats_partial_kernel<uint16_t><<<nblocks, 256, 0, s>>>((const uint16_t*)W, n_elems / 8, partials);
  PQ_CHECK_LAUNCH("wstats_partial_kernel");
  return PQ_OK;
}

template <typename T, bool RAGGED>
__global__ __launch_bounds__(256) void pack_sign_kernel(const T* __restrict__ W, int N, int K,
                                                        const double* __restrict__ partials, int G,
                                                        uint8_t* __restrict__ Pbytes,
                                                        uint32_t* __restrict__ Pt,
                                                        float* __restrict__ mu_lambda) {
  pack_sign_body<T, RAGGED>(W, N, K, partials, G, Pbytes, Pt, mu_lambda, blockIdx.x, blockIdx.y);
}
// one bf16 weight, and behind its tiles the rows of two small matrices on the AbsMax grid (the factors of the INT8 branch: two
// launches of about 5 us less)
__global__ __launch_bounds__(256) void pack_quant_rows_kernel(const uint16_t* __restrict__ W, int N, int K, const double* __restrict__ partials,
                                                              int G, uint8_t* __restrict__ Pbytes, uint32_t* __restrict__ Pt,
                                                              float* __restrict__ mu_lambda, int gx, int npack, pq_quant_rows_job j0,
                                                              pq_quant_rows_job j1) {
  int b = blockIdx.x;
  if (b < npack) {                                   // uniform (N and K are whole words here)
    pack_sign_body<uint16_t, false>(W, N, K, partials, G, Pbytes, Pt, mu_lambda, b % gx, b / gx);
    return;
  }
  b -= npack;
  const int n0 = (j0.rows + 3) / 4;
  const pq_quant_rows_job& j = b < n0 ? j0 : j1;
  quant_act_body<uint16_t, 0>((const uint16_t*)j.src, j.rows, j.cols, j.codes, j.gamma, j.deq, b < n0 ? b : b - n0);
}
int pq_launch_pack_quant_rows(const void* W, int N, int K, const double* partials, int nblocks, uint32_t* P, uint32_t* Pt, float* mu_lambda,
                              const pq_quant_rows_job* jobs, hipStream_t s) {
  if (N % 32 != 0 || K % 32 != 0) return pq_set_error(PQ_ERR_SHAPE, "N=%d and K=%d must be multiples of 32", N, K);
  pq_prof_scope prof(PQP_PACK, s);
  const int gx = (K + 511) / 512, npack = gx * (N / 32);
  const int nrow = (jobs[0].rows + 3) / 4 + (jobs[1].rows + 3) / 4;
  pack_quant_rows_kernel<<<npack + nrow, 256, 0, s>>>((const uint16_t*)W, N, K, partials, nblocks, (uint8_t*)P, Pt, mu_lambda, gx, npack, jobs[0], jobs[1]);
  PQ_CHECK_LAUNCH("pack_quant_rows_kernel");
  return PQ_OK;
}
// one bf16 weight (npack workgroups, none where it is packed already) behind the ordering of a routed call's slots
__global__ __launch_bounds__(256) void pack_place_kernel(const uint16_t* __restrict__ W, int N, int K, const double* __restrict__ partials,
                                                         int G, uint8_t* __restrict__ Pbytes, uint32_t* __restrict__ Pt,
                                                         float* __restrict__ mu_lambda, int gx, pq_place place, int groups, int subs) {
  const int b = blockIdx.x;
  const int np = groups * subs;
  if (b < np) {                                      // uniform
    place_body(place, b, groups, subs);
    return;
  }
  pack_sign_body<uint16_t, false>(W, N, K, partials, G, Pbytes, Pt, mu_lambda, (b - np) % gx, (b - np) / gx);
}
int pq_launch_pack_place(const void* W, int N, int K, const double* partials, int nblocks, uint32_t* P, uint32_t* Pt, float* mu_lambda,
                         const pq_place& place, hipStream_t s) {
  if (N % 32 != 0 || K % 32 != 0) return pq_set_error(PQ_ERR_SHAPE, "N=%d and K=%d must be multiples of 32", N, K);
  pq_prof_scope prof(W ? PQP_PACK : PQP_MOE_ROUTE, s);
  const int gx = (K + 511) / 512, groups = place_groups(place.nblk), subs = place_subs(place.nblk);
  pack_place_kernel<<<groups * subs + (W ? gx * (N / 32) : 0), 256, 0, s>>>((const uint16_t*)W, N, K, partials, nblocks, (uint8_t*)P, Pt, mu_lambda, gx, place,
                                                                          groups, subs);
  PQ_CHECK_LAUNCH("pack_place_kernel");
  return PQ_OK;
}
// three bf16 weights in one launch, the tiles of one after those of the other (PLACE: behind the ordering of the slots)
struct pack3_args { pq_weight_job w[3]; pq_place place; int groups, subs; };
template <bool RAGGED, bool PLACE>
__global__ __launch_bounds__(256) void pack_sign3_kernel(pack3_args a) {
  int b = blockIdx.x, i = 0;
  if constexpr (PLACE) {
    if (b < a.groups * a.subs) {                     // uniform
      place_body(a.place, b, a.groups, a.subs);
      return;
    }
    b -= a.groups * a.subs;
  }
  int gx = (((a.w[0].K + 31) & ~31) + 511) / 512, n = gx * ((a.w[0].N + 31) / 32);
  while (i < 2 && b >= n) {                          // uniform
    b -= n;
    ++i;
    gx = (((a.w[i].K + 31) & ~31) + 511) / 512;
    n = gx * ((a.w[i].N + 31) / 32);
  }
  const pq_weight_job& w = a.w[i];
  pack_sign_body<uint16_t, RAGGED>((const uint16_t*)w.W, w.N, w.K, w.partials, w.nblocks, (uint8_t*)w.P, w.Pt, w.mu_lambda, b % gx, b / gx);
}
int pq_launch_pack3(const pq_weight_job* w, const pq_place* place, hipStream_t s) {
  pq_prof_scope prof(PQP_PACK, s);
  pack3_args a;
  memset(&a, 0, sizeof(a));
  bool ragged = false;
  unsigned blocks = 0;
  if (place) {
    a.place = *place;
    a.groups = place_groups(place->nblk);
    a.subs = place_subs(place->nblk);
    blocks = (unsigned)(a.groups * a.subs);
  }
  for (int i = 0; i < 3; ++i) {
    a.w[i] = w[i];
    ragged = ragged || w[i].K % 32 || w[i].N % 32;
    blocks += (unsigned)((((w[i].K + 31) & ~31) + 511) / 512) * ((w[i].N + 31) / 32);
  }
  if (place) {
    if (ragged) pack_sign3_kernel<true, true><<<blocks, 256, 0, s>>>(a);
    else pack_sign3_kernel<false, true><<<blocks, 256, 0, s>>>(a);
  } else if (ragged) pack_sign3_kernel<true, false><<<blocks, 256, 0, s>>>(a);
  else pack_sign3_kernel<false, false><<<blocks, 256, 0, s>>>(a);
  PQ_CHECK_LAUNCH("pack_sign3_kernel");
  return PQ_OK;
}

int pq_launch_pack(const void* W, int dtype, int N, int K, const double* partials, int nblocks,
                   uint32_t* P, uint32_t* Pt, float* mu_lambda, hipStream_t s) {
  pq_prof_scope prof(PQP_PACK, s);
  const int Kp = (K + 31) & ~31;
  dim3 grid((Kp + 511) / 512, (N + 31) / 32), block(256);
  const bool ragged = (K % 32 != 0) || (N % 32 != 0);
  if (dtype == PQ_F32) {
    if (ragged) pack_sign_kernel<float, true><<<grid, block, 0, s>>>((const float*)W, N, K, partials, nblocks, (uint8_t*)P, Pt, mu_lambda);
    else pack_sign_kernel<float, false><<<grid, block, 0, s>>>((const float*)W, N, K, partials, nblocks, (uint8_t*)P, Pt, mu_lambda);
  } else {
    if (ragged) pack_sign_kernel<uint16_t, true><<<grid, block, 0, s>>>((const uint16_t*)W, N, K, partials, nblocks, (uint8_t*)P, Pt, mu_lambda);
    else pack_sign_kernel<uint16_t, false><<<grid, block, 0, s>>>((const uint16_t*)W, N, K, partials, nblocks, (uint8_t*)P, Pt, mu_lambda);
  }
  PQ_CHECK_LAUNCH("pack_sign_kernel");
  return PQ_OK;
}

template <typename T>
static int launch_router_t(const T* X, const T* Wr, int Tn, int K, int E, int k, int* idx, float* gate,
                           float* probs, hipStream_t s, int* hist) {
  const dim3 block(256), grid((Tn + pq_router_tokens(E) - 1) / pq_router_tokens(E));
  if (E <= 8) router_kernel<T, 8, 4><<<grid, block, 0, s>>>(X, Wr, Tn, K, E, k, idx, gate, probs, hist);
  else if (E <= 16) router_kernel<T, 16, 2><<<grid, block, 0, s>>>(X, Wr, Tn, K, E, k, idx, gate, probs, hist);
  else router_kernel<T, 64, 1><<<grid, block, 0, s>>>(X, Wr, Tn, K, E, k, idx, gate, probs, hist);
  PQ_CHECK_LAUNCH("router_kernel");
  return PQ_OK;
}

int pq_launch_router(const void* X, const void* Wr, int dtype, int T, int K, int E, int k, int* idx,
                     float* gate, float* probs, hipStream_t s, int* hist) {
  if (T == 0) return PQ_OK;
  pq_prof_scope prof(PQP_ROUTER, s);
  if (dtype == PQ_F32)
    return launch_router_t<float>((const float*)X, (const float*)Wr, T, K, E, k, idx, gate, probs, s, hist);
  return launch_router_t<uint16_t>((const uint16_t*)X, (const uint16_t*)Wr, T, K, E, k, idx, gate, probs, s, hist);
}

// ------------------------------------------------------------------------------------------
// Fixed-order final reduction of per-block partial sums.
// ------------------------------------------------------------------------------------------
typedef pq_reduce_job reduce_job;

__global__ __launch_bounds__(256) void reduce_partials_kernel(reduce_job j0, reduce_job j1) {   // one workgroup per job
  pq_reduce_job_body(blockIdx.x == 0 ? j0 : j1);
}

// two independent reductions in one launch
int pq_launch_reduce_partials2(const double* pa, int na, float fa, const float* dfa, float* oa, const double* pb, int nb, float fb,
                               const float* dfb, float* ob, hipStream_t s) {
  pq_prof_scope prof(PQP_REDUCE, s);
  reduce_partials_kernel<<<2, 256, 0, s>>>(reduce_job{pa, na, fa, dfa, oa}, reduce_job{pb, nb, fb, dfb, ob});
  PQ_CHECK_LAUNCH("reduce_partials_kernel");
  return PQ_OK;
}
