// Element-wise kernels of the decoupled FFN and the routed experts (Sec. 3.2, 3.3): row gather, the gated unit with fused AbsMax re-quantisation,
// expert activation forward/backward, gate/alpha reductions, router backward, scatter-combine.
// All tensors here are bf16 unless noted; every reduction has a fixed order.
#include "pq_epilogue.h"

namespace {

__device__ __forceinline__ void unpack8(const uint4& u, float* f) {
  f[0] = __uint_as_float(u.x << 16); f[1] = __uint_as_float(u.x & 0xFFFF0000u);
  f[2] = __uint_as_float(u.y << 16); f[3] = __uint_as_float(u.y & 0xFFFF0000u);
  f[4] = __uint_as_float(u.z << 16); f[5] = __uint_as_float(u.z & 0xFFFF0000u);
  f[6] = __uint_as_float(u.w << 16); f[7] = __uint_as_float(u.w & 0xFFFF0000u);
}
__device__ __forceinline__ uint4 pack8(const float* f) {
  return make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7]));
}
__device__ __forceinline__ float dsiluf_(float x) {
  const float s = pq_sigmoid(x);
  return s * (1.0f + x * (1.0f - s));
}

// dst[pos][:] = src[perm[pos] / k][:]   (rows of d bf16, d % 8 == 0), one wavefront per row
__global__ __launch_bounds__(256) void gather_rows_kernel(const uint16_t* __restrict__ src, const int* __restrict__ perm, int k,
                                                          int S, int d, uint16_t* __restrict__ dst) {
  const int pos = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (pos >= S) return;
  const int t = perm[pos] / k;
  const uint4* s4 = reinterpret_cast<const uint4*>(src + (size_t)t * d);
  uint4* d4 = reinterpret_cast<uint4*>(dst + (size_t)pos * d);
  for (int c = lane; c < d / 8; c += 64) d4[c] = s4[c];
}

// ---- the gated unit with fused AbsMax re-quantisation (one wavefront per token) -------------
//   Hd = silu(G) * U in fp32; gamma_h = 128 / max(|Hd|, 1e-5); Hq = codes; Ht = bf16(Hq / gamma_h)
// Rows are F elements apart; only the first Fv columns exist (Fv % 4 == 0): the others are written as zero codes,
// whatever U and G hold there (a width that is not a multiple of 32 is padded, Table 1: 5076 -> 5088).
// All of a row's vectors are requested before the first is used, so a token costs one memory latency.
template <int NV>
__global__ __launch_bounds__(256) void swiglu_quant_kernel(const uint16_t* __restrict__ U, const uint16_t* __restrict__ G,
                                                           int T, int F, int Fv, int8_t* __restrict__ Hq, float* __restrict__ gamma,
                                                           uint16_t* __restrict__ Ht) {
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (t >= T) return;
  const uint4* u4 = reinterpret_cast<const uint4*>(U + (size_t)t * F);
  const uint4* g4 = reinterpret_cast<const uint4*>(G + (size_t)t * F);
  const int nvec = F / 8;
  float hd[NV > 0 ? NV : 1][8];
  float amax = 0.0f;
  auto gated = [&](const uint4& u, const uint4& g, int c, float* h) {
    float uf[8], gf[8];
    unpack8(u, uf);
    unpack8(g, gf);
#pragma unroll
    for (int j = 0; j < 8; ++j) h[j] = (c * 8 + j < Fv) ? pq_silu(gf[j]) * uf[j] : 0.0f;
  };
  if constexpr (NV > 0) {
    uint4 ur[NV], gr[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      // unconditional (lanes past the end repeat the last vector, which cannot change the maximum): loads under
      // a branch would each get a wait of their own
      const int c = min(i * 64 + lane, nvec - 1);
      ur[i] = u4[c];
      gr[i] = g4[c];
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      gated(ur[i], gr[i], min(i * 64 + lane, nvec - 1), hd[i]);
#pragma unroll
      for (int j = 0; j < 8; ++j) amax = fmaxf(amax, fabsf(hd[i][j]));
    }
  } else {
    for (int c = lane; c < nvec; c += 64) {
      float h[8];
      gated(u4[c], g4[c], c, h);
#pragma unroll
      for (int j = 0; j < 8; ++j) amax = fmaxf(amax, fabsf(h[j]));
    }
  }
  amax = wave_max(amax);
  const float g = 128.0f / fmaxf(amax, 1e-5f);
  const float ginv = 1.0f / g;                       // q / gamma as q * (1 / gamma): one division per token
  if (lane == 0) gamma[t] = g;
  auto emit = [&](int c, const float* h) {
    int q[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) q[j] = (int)fminf(fmaxf(rintf(__fmul_rn(h[j], g)), -128.0f), 127.0f);
    const uint32_t w0 = (uint32_t)(q[0] & 0xFF) | ((uint32_t)(q[1] & 0xFF) << 8) | ((uint32_t)(q[2] & 0xFF) << 16) | ((uint32_t)(q[3] & 0xFF) << 24);
    const uint32_t w1 = (uint32_t)(q[4] & 0xFF) | ((uint32_t)(q[5] & 0xFF) << 8) | ((uint32_t)(q[6] & 0xFF) << 16) | ((uint32_t)(q[7] & 0xFF) << 24);
    *reinterpret_cast<uint2*>(Hq + (size_t)t * F + (size_t)c * 8) = make_uint2(w0, w1);
    float o[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j] = __fmul_rn((float)q[j], ginv);
    *reinterpret_cast<uint4*>(Ht + (size_t)t * F + (size_t)c * 8) = pack8(o);
  };
  if constexpr (NV > 0) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c = i * 64 + lane;
      if (c < nvec) emit(c, hd[i]);
    }
  } else {
    for (int c = lane; c < nvec; c += 64) {
      float h[8];
      gated(u4[c], g4[c], c, h);
      emit(c, h);
    }
  }
}

// dU = dHd * silu(G), dG = dHd * U * silu'(G)   (element-wise over rows of F elements of which the first Fv exist; the
// others are written as zeros; two vectors of 8 per thread and pass)
__global__ __launch_bounds__(256) void swiglu_bwd_kernel(const uint16_t* __restrict__ dHd, const uint16_t* __restrict__ U,
                                                         const uint16_t* __restrict__ G, size_t nvec, int F, int Fv,
                                                         uint16_t* __restrict__ dU, uint16_t* __restrict__ dG) {
  const size_t stride = (size_t)gridDim.x * 256;
  const int vpr = F / 8;                             // vectors per row
  for (size_t c0 = (size_t)blockIdx.x * 256 + threadIdx.x; c0 < nvec; c0 += 2 * stride) {
    const size_t c1 = c0 + stride;
    const bool two = c1 < nvec;
    const size_t cb = two ? c1 : c0;
    const uint4 r0[3] = {reinterpret_cast<const uint4*>(dHd)[c0], reinterpret_cast<const uint4*>(U)[c0], reinterpret_cast<const uint4*>(G)[c0]};
    const uint4 r1[3] = {reinterpret_cast<const uint4*>(dHd)[cb], reinterpret_cast<const uint4*>(U)[cb], reinterpret_cast<const uint4*>(G)[cb]};
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (q == 1 && !two) break;
      const size_t c = q ? c1 : c0;
      const int col = (int)(c % (size_t)vpr) * 8;
      uint4 du, dg;
      pq_swiglu_bwd8(q ? r1[0] : r0[0], q ? r1[1] : r0[1], q ? r1[2] : r0[2], col, Fv, du, dg);
      reinterpret_cast<uint4*>(dU)[c] = du;
      reinterpret_cast<uint4*>(dG)[c] = dg;
    }
  }
}

// ---- expert activation ----------------------------------------------------------------------
// a = silu(ge) * ue  over S rows of r elements (slot order); ue and ge have a row stride of ld elements (r, or 2 r when
// both lie side by side in one [S][2 r] product)
__global__ __launch_bounds__(256) void expert_act_kernel(const uint16_t* __restrict__ ue, const uint16_t* __restrict__ ge,
                                                         int ld, int r, size_t nvec, uint16_t* __restrict__ a) {
  const size_t c = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (c >= nvec) return;
  const size_t pos = c / (size_t)(r / 8), in = pos * ld + (c - pos * (size_t)(r / 8)) * 8;
  float uf[8], gf[8], o[8];
  unpack8(*reinterpret_cast<const uint4*>(ue + in), uf);
  unpack8(*reinterpret_cast<const uint4*>(ge + in), gf);
#pragma unroll
  for (int j = 0; j < 8; ++j) o[j] = pq_silu(gf[j]) * uf[j];
  reinterpret_cast<uint4*>(a)[c] = pack8(o);
}

// with s = alpha * gate[slot] (perm == NULL: a single branch, s = alpha):  du = s da silu(ge), dg = s da ue silu'(ge), as = s a
// (r % 8 == 0).  The first `ride` workgroups of a single branch's launch form d alpha and d beta and clear dWr, which no gradient
// reaches: a launch of its own took 4.6 us at the end of every backward.
__global__ __launch_bounds__(256) void expert_act_bwd_kernel(const uint16_t* __restrict__ da, const uint16_t* __restrict__ ue,
                                                             const uint16_t* __restrict__ ge, const uint16_t* __restrict__ a,
                                                             const int* __restrict__ perm, const float* __restrict__ gate,
                                                             float alpha, int r, int ld, size_t nvec, uint16_t* __restrict__ du,
                                                             uint16_t* __restrict__ dg, uint16_t* __restrict__ as, int ride,
                                                             float* __restrict__ dWr, int n_wr, pq_reduce_job j0, pq_reduce_job j1) {
  if ((int)blockIdx.x < ride) {                      // uniform
    if (blockIdx.x < 2) pq_reduce_job_body(blockIdx.x == 0 ? j0 : j1);
    else if (const int i = (blockIdx.x - 2) * 256 + threadIdx.x; i < n_wr) dWr[i] = 0.0f;
    return;
  }
  const size_t c = (size_t)(blockIdx.x - ride) * 256 + threadIdx.x;
  if (c >= nvec) return;
  const int pos = (int)(c / (size_t)(r / 8));
  const size_t in = (size_t)pos * ld + (c - (size_t)pos * (r / 8)) * 8;   // ue, ge, du, dg: row stride ld (r or 2 r)
  const float sc = perm ? alpha * gate[perm[pos]] : alpha;
  float d[8], uf[8], gf[8], af[8], o1[8], o2[8], o3[8];
  unpack8(reinterpret_cast<const uint4*>(da)[c], d);
  unpack8(*reinterpret_cast<const uint4*>(ue + in), uf);
  unpack8(*reinterpret_cast<const uint4*>(ge + in), gf);
  unpack8(reinterpret_cast<const uint4*>(a)[c], af);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float dj = sc * d[j];           // upstream of the expert output is alpha * gate * dY
    o1[j] = dj * pq_silu(gf[j]);
    o2[j] = dj * uf[j] * dsiluf_(gf[j]);
    o3[j] = sc * af[j];
  }
  *reinterpret_cast<uint4*>(du + in) = pack8(o1);
  *reinterpret_cast<uint4*>(dg + in) = pack8(o2);
  reinterpret_cast<uint4*>(as)[c] = pack8(o3);
}

// One pass over the upstream gradient in slot order: rd[pos] = <dY[t], Ys[pos]> (fp32) with t = perm[pos] / k,
// partial[block] = sum gate[perm[pos]] * rd[pos] (for d alpha), and dst[pos] = dY[t], with SCALE times
// alpha * gate (the upstream gradient of an expert's output).  perm NULL: a single branch (slot pos is token pos, gate 1), of
// which the sum alone is wanted: gate, rd and dst are NULL too.  Gather, dot and scaling in passes of their own read and wrote
// the slot rows three times: routed linear of 1531 tokens 1056 -> 3104, two experts each, 6.9 + 8.2 + 6.8 us.
template <bool SCALE>
__global__ __launch_bounds__(256) void slot_grad_kernel(const uint16_t* __restrict__ dY, const uint16_t* __restrict__ Ys,
                                                        const int* __restrict__ perm, const float* __restrict__ gate, float alpha, int k,
                                                        int S, int d, uint16_t* __restrict__ dst, float* __restrict__ rd,
                                                        double* __restrict__ partial) {
  __shared__ double red[4];
  const int pos = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  double contrib = 0.0;
  if (pos < S) {
    const int slot = perm ? perm[pos] : pos;
    const float gt = perm ? gate[slot] : 1.0f, sc = alpha * gt;
    const uint4* a4 = reinterpret_cast<const uint4*>(dY + (size_t)(slot / k) * d);
    const uint4* b4 = reinterpret_cast<const uint4*>(Ys + (size_t)pos * d);
    uint4* o4 = reinterpret_cast<uint4*>(dst + (size_t)pos * d);
    const int n = d / 8;
    float acc = 0.0f;
    for (int cb = lane; cb < n; cb += 256) {          // eight loads in flight (past the end: the last vector, dropped)
      uint4 a[4], b[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = min(cb + 64 * q, n - 1);
        a[q] = a4[c];
        b[q] = b4[c];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = cb + 64 * q;
        if (c >= n) break;
        float x[8], y[8];
        unpack8(a[q], x);
        unpack8(b[q], y);
#pragma unroll
        for (int j = 0; j < 8; ++j) acc += x[j] * y[j];
        if (dst) {                                    // uniform
          if constexpr (SCALE) {
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] *= sc;
            o4[c] = pack8(x);
          } else o4[c] = a[q];
        }
      }
    }
    acc = wave_sum(acc);
    if (lane == 0) {
      if (rd) rd[pos] = acc;
      contrib = (double)gt * (double)acc;
    }
  }
  const double t = block_sum_d<256>(contrib, red);
  if (threadIdx.x == 0) partial[blockIdx.x] = t;
}

// Y[t,:] += alpha * sum_j gate[t,j] * Ys[inv[t*k+j], :]   (one wavefront per token)
__global__ __launch_bounds__(256) void combine_fwd_kernel(uint16_t* __restrict__ Y, const uint16_t* __restrict__ Ys,
                                                          const int* __restrict__ inv, const float* __restrict__ gate, float alpha,
                                                          int T, int k, int d) {
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (t >= T) return;
  uint4* y4 = reinterpret_cast<uint4*>(Y + (size_t)t * d);
  const int n = d / 8;
  // four vectors of Y and of two slots in flight (past the end: the last vector, dropped); one at a time it was a chain of memory
  // latencies (1531 tokens, 3104 columns, two slots each: 14 us, now 8)
  for (int cb = lane; cb < n; cb += 256) {
    uint4 yv[4];
    float acc[4][8];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      yv[q] = y4[min(cb + 64 * q, n - 1)];
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[q][i] = 0.0f;
    }
    for (int j = 0; j < k; j += 2) {
      const int j1 = min(j + 1, k - 1);
      const float g0 = gate[t * k + j], g1 = gate[t * k + j1];
      const uint4* s0 = reinterpret_cast<const uint4*>(Ys + (size_t)inv[t * k + j] * d);
      const uint4* s1 = reinterpret_cast<const uint4*>(Ys + (size_t)inv[t * k + j1] * d);
      uint4 a[4], b[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) a[q] = s0[min(cb + 64 * q, n - 1)];
      if (j + 1 < k) {                                // uniform
#pragma unroll
        for (int q = 0; q < 4; ++q) b[q] = s1[min(cb + 64 * q, n - 1)];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float v[8];
        unpack8(a[q], v);
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[q][i] += g0 * v[i];
      }
      if (j + 1 < k) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float v[8];
          unpack8(b[q], v);
#pragma unroll
          for (int i = 0; i < 8; ++i) acc[q][i] += g1 * v[i];
        }
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (cb + 64 * q >= n) break;
      float y[8];
      unpack8(yv[q], y);
#pragma unroll
      for (int i = 0; i < 8; ++i) y[i] += alpha * acc[q][i];
      y4[cb + 64 * q] = pack8(y);
    }
  }
}

// dlogit[t,e] = sum_j dgate[t,j] * p[idx_j] * (1[e == idx_j] - p[e]),  dgate[t,j] = alpha * rd[inv[t*k+j]]
__device__ __forceinline__ float router_dlogit(const float* __restrict__ rd, const int* __restrict__ inv, const int* __restrict__ idx,
                                               const float* __restrict__ probs, float alpha, int k, int E, int t, int e) {
  const float pe = probs[(size_t)t * E + e];
  float acc = 0.0f;
  for (int j = 0; j < k; ++j) {
    const int ej = idx[t * k + j];
    const float dgt = alpha * rd[inv[t * k + j]];
    acc += dgt * probs[(size_t)t * E + ej] * ((e == ej ? 1.0f : 0.0f) - pe);
  }
  return acc;
}

// Tokens to a chunk: 128, or 32 while 128 leave CUs without a workgroup (1531 tokens, 1056 columns, four experts: 60 workgroups
// 18 us, 240 of them 6; 8192 tokens, 2048 columns: 128 20 us, 32 27).
int dwr_chunk(int T, int d) { return ((d + 255) / 256) * ((T + 127) / 128) < 256 ? 32 : 128; }

// dWr partials: part[tc][e][c] = sum_{t in chunk tc} dlogit[t,e] * X[t,c].
// A workgroup covers 256 columns of one chunk: thread = (token subgroup sg, column group cg); it walks every
// eighth token t0 + sg, t0 + sg + 8, ... with 16-byte loads of 8 columns, then the 8 subgroups are summed in LDS
// in a fixed order.
// dlogit is formed here, by every column block for itself; the first one leaves it in memory for the input gradient.
template <int DWR_CHUNK>
__global__ __launch_bounds__(256) void dwr_partial_kernel(const float* __restrict__ rd, const int* __restrict__ inv, const int* __restrict__ idx,
                                                          const float* __restrict__ probs, float alpha, int k, float* __restrict__ dlogit,
                                                          const uint16_t* __restrict__ X, int T, int d, int E, float* __restrict__ part) {
  __shared__ float red[8][4][8][32];                 // [subgroup][expert % 4][column % 8][column group]
  __shared__ __attribute__((aligned(16))) float sdl[DWR_CHUNK][8];   // the chunk's dlogit for the eight experts of a pass (zero past E and past T)
  const int tid = threadIdx.x, cg = tid & 31, sg = tid >> 5;
  const int c0 = blockIdx.x * 256 + cg * 8;
  const int t0 = blockIdx.y * DWR_CHUNK;
  const bool okc = c0 < d;                            // d % 8 == 0
  for (int e0 = 0; e0 < E; e0 += 8) {
    // every load below is unconditional (indices clamped into the arrays, the value masked afterwards): a load under
    // a branch waits for its own latency, and the loop over tokens becomes a chain of them
    for (int o = tid; o < DWR_CHUNK * 8; o += 256) {
      const int tt = o >> 3, u = o & 7;
      const int t = min(t0 + tt, T - 1), e = min(e0 + u, E - 1);
      const float g = router_dlogit(rd, inv, idx, probs, alpha, k, E, t, e);
      const bool in = t0 + tt < T && e0 + u < E;
      sdl[tt][u] = in ? g : 0.0f;
      if (in && blockIdx.x == 0) dlogit[(size_t)t * E + e] = g;
    }
    __syncthreads();
    float acc[8][8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[u][j] = 0.0f;
    if (okc) {
      constexpr int Q = DWR_CHUNK < 64 ? DWR_CHUNK / 8 : 8;
      for (int grp = 0; grp < DWR_CHUNK / (8 * Q); ++grp) {   // Q of the subgroup's tokens at a time, their loads issued together
        uint4 xv[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q)
          xv[q] = *reinterpret_cast<const uint4*>(X + (size_t)min(t0 + sg + 8 * (Q * grp + q), T - 1) * d + c0);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const int tt = sg + 8 * (Q * grp + q);
          const float4 ga = *reinterpret_cast<const float4*>(&sdl[tt][0]), gb = *reinterpret_cast<const float4*>(&sdl[tt][4]);
          const float g[8] = {ga.x, ga.y, ga.z, ga.w, gb.x, gb.y, gb.z, gb.w};
          float x[8];
          unpack8(xv[q], x);
#pragma unroll
          for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[u][j] += g[u] * x[j];
        }
      }
    }
#pragma unroll
    for (int half = 0; half < 2; ++half) {           // four experts per round through LDS
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int j = 0; j < 8; ++j) red[sg][u][j][cg] = acc[4 * half + u][j];
      __syncthreads();
      for (int o = tid; o < 4 * 256; o += 256) {
        const int u = o >> 8, c = o & 255, e = e0 + 4 * half + u;
        if (e < E && blockIdx.x * 256 + c < d) {
          float v = 0.0f;
#pragma unroll
          for (int q = 0; q < 8; ++q) v += red[q][u][c & 7][c >> 3];
          part[((size_t)blockIdx.y * E + e) * d + blockIdx.x * 256 + c] = v;
        }
      }
      __syncthreads();
    }
  }
}
// dWr = the chunks' partial sums added in chunk order (eight loads in flight per thread; no chunks: zeros).  Two scalar
// reductions of the same call (d alpha, d beta) ride along as the last workgroups.
__global__ __launch_bounds__(256) void dwr_final_kernel(const float* __restrict__ part, int nchunks, int n, float* __restrict__ dWr,
                                                        pq_reduce_job j0, pq_reduce_job j1) {
  const int nb = (n + 255) / 256;
  if ((int)blockIdx.x >= nb) {                       // uniform
    pq_reduce_job_body((int)blockIdx.x == nb ? j0 : j1);
    return;
  }
  const int i = blockIdx.x * 256 + threadIdx.x;   // e * d + c
  if (i >= n) return;
  float acc = 0.0f;
  for (int tc = 0; tc < nchunks; tc += 8) {
    float v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = part[(size_t)min(tc + q, nchunks - 1) * n + i];
#pragma unroll
    for (int q = 0; q < 8; ++q) acc += (tc + q < nchunks) ? v[q] : 0.0f;
  }
  dWr[i] = acc;
}

// dX[t,:] += sum_j dXs[inv[t*k+j], :] + sum_e dlogit[t,e] * Wr[e,:]
__global__ __launch_bounds__(256) void combine_bwd_kernel(uint16_t* __restrict__ dX, const uint16_t* __restrict__ dXs,
                                                          const int* __restrict__ inv, const float* __restrict__ dlogit,
                                                          const uint16_t* __restrict__ Wr, int T, int k, int d, int E) {
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (t >= T) return;
  uint4* x4 = reinterpret_cast<uint4*>(dX + (size_t)t * d);
  const int n = d / 8;
  // four vectors of a row in flight (past the end: the last vector, dropped), and the next row's while one is added
  for (int cb = lane; cb < n; cb += 256) {
    float acc[4][8];
    uint4 x[4], w[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = x4[min(cb + 64 * q, n - 1)];
    const int rows = k + E;                           // the slots' rows, then the router's
    auto row = [&](int j) { return reinterpret_cast<const uint4*>(j < k ? dXs + (size_t)inv[t * k + j] * d : Wr + (size_t)(j - k) * d); };
    auto fetch = [&](int j) {
      const uint4* r = row(j);
#pragma unroll
      for (int q = 0; q < 4; ++q) w[q] = r[min(cb + 64 * q, n - 1)];
    };
    fetch(0);
#pragma unroll
    for (int q = 0; q < 4; ++q) unpack8(x[q], acc[q]);
    for (int j = 0; j < rows; ++j) {
      const float f = j < k ? 1.0f : dlogit[(size_t)t * E + j - k];
      float v[4][8];
#pragma unroll
      for (int q = 0; q < 4; ++q) unpack8(w[q], v[q]);
      fetch(min(j + 1, rows - 1));
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[q][i] += f * v[q][i];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (cb + 64 * q < n) x4[cb + 64 * q] = pack8(acc[q]);
  }
}

// The same with the router matrix in LDS (E * d bf16 <= 64 KB, E <= 64) and a token's pieces requested together: NC
// 16-byte pieces per lane (d = 512 NC), up to KMAX slots per token; lane e fetches dlogit[t][e] once and hands it round.
// A workgroup takes CB_TOK tokens per wavefront, so the router matrix is staged once
// per 4 * CB_TOK tokens.  Same sums in the same order as above.
constexpr int CB_TOK = 4;
template <int NC, int KMAX>
__global__ __launch_bounds__(256) void combine_bwd_lds_kernel(uint16_t* __restrict__ dX, const uint16_t* __restrict__ dXs,
                                                              const int* __restrict__ inv, const float* __restrict__ dlogit,
                                                              const uint16_t* __restrict__ Wr, int T, int k, int E) {
  extern __shared__ __attribute__((aligned(16))) unsigned char wr_s[];   // [E][d] bf16
  constexpr int d = 512 * NC;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  {
    const int nvec = E * d / 8;
    for (int c = threadIdx.x; c < nvec; c += 256) reinterpret_cast<uint4*>(wr_s)[c] = reinterpret_cast<const uint4*>(Wr)[c];
  }
  __syncthreads();
  for (int q = 0; q < CB_TOK; ++q) {
    const int t = (blockIdx.x * 4 + wave) * CB_TOK + q;
    if (t >= T) break;                                // wave-uniform
    int pos[KMAX];
#pragma unroll
    for (int j = 0; j < KMAX; ++j) pos[j] = inv[t * k + min(j, k - 1)];
    const float dlv = lane < E ? dlogit[(size_t)t * E + lane] : 0.0f;
    uint4* x4 = reinterpret_cast<uint4*>(dX + (size_t)t * d) + lane;
    uint4 xv[NC], sv[KMAX][NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) xv[i] = x4[64 * i];
#pragma unroll
    for (int j = 0; j < KMAX; ++j)
#pragma unroll
      for (int i = 0; i < NC; ++i) sv[j][i] = reinterpret_cast<const uint4*>(dXs + (size_t)pos[j] * d)[lane + 64 * i];
    float acc[NC][8];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      unpack8(xv[i], acc[i]);
#pragma unroll
      for (int j = 0; j < KMAX; ++j) {
        if (j < k) {
          float v[8];
          unpack8(sv[j][i], v);
#pragma unroll
          for (int u = 0; u < 8; ++u) acc[i][u] += v[u];
        }
      }
    }
    for (int e = 0; e < E; ++e) {
      const float dl = __shfl(dlv, e);
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        float w[8];
        unpack8(reinterpret_cast<const uint4*>(wr_s + (size_t)e * d * 2)[lane + 64 * i], w);
#pragma unroll
        for (int u = 0; u < 8; ++u) acc[i][u] += dl * w[u];
      }
    }
#pragma unroll
    for (int i = 0; i < NC; ++i) x4[64 * i] = pack8(acc[i]);
  }
}

// out = sum_i c[i] * x[i]  (up to 4 bf16 tensors, fp32 arithmetic, one rounding): the glue between
// the linears of a layer stack (residual adds, the stand-in for the attention core)
__global__ __launch_bounds__(256) void lincomb_kernel(uint16_t* __restrict__ out, const uint16_t* x0, const uint16_t* x1,
                                                      const uint16_t* x2, const uint16_t* x3, float c0, float c1, float c2,
                                                      float c3, size_t nvec) {
  for (size_t c = (size_t)blockIdx.x * 256 + threadIdx.x; c < nvec; c += (size_t)gridDim.x * 256) {
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0}, v[8];
    unpack8(reinterpret_cast<const uint4*>(x0)[c], v);
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = c0 * v[j];
    if (x1) {
      unpack8(reinterpret_cast<const uint4*>(x1)[c], v);
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[j] += c1 * v[j];
    }
    if (x2) {
      unpack8(reinterpret_cast<const uint4*>(x2)[c], v);
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[j] += c2 * v[j];
    }
    if (x3) {
      unpack8(reinterpret_cast<const uint4*>(x3)[c], v);
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[j] += c3 * v[j];
    }
    reinterpret_cast<uint4*>(out)[c] = pack8(acc);
  }
}

}  // namespace

int pq_launch_lincomb(void* out, const void* x0, const void* x1, const void* x2, const void* x3, float c0, float c1, float c2,
                      float c3, size_t n, hipStream_t s) {
  if (n == 0) return PQ_OK;
  pq_prof_scope prof(PQP_GLUE, s);
  const size_t nvec = n / 8;
  size_t blocks = (nvec + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  lincomb_kernel<<<(unsigned)blocks, 256, 0, s>>>((uint16_t*)out, (const uint16_t*)x0, (const uint16_t*)x1, (const uint16_t*)x2,
                                                 (const uint16_t*)x3, c0, c1, c2, c3, nvec);
  PQ_CHECK_LAUNCH("lincomb_kernel");
  return PQ_OK;
}

// ---------------------------------------------------------------------------------------------
int pq_launch_gather_rows(const void* src, const int* perm, int k, int S, int d, void* dst, hipStream_t s) {
  if (S == 0) return PQ_OK;
  pq_prof_scope prof(PQP_MOE_ELEMENTWISE, s);
  gather_rows_kernel<<<(S + 3) / 4, 256, 0, s>>>((const uint16_t*)src, perm, k, S, d, (uint16_t*)dst);
  PQ_CHECK_LAUNCH("gather_rows_kernel");
  return PQ_OK;
}

int pq_launch_swiglu_quant(const void* U, const void* G, int T, int F, int Fv, int8_t* Hq, float* gamma, void* Ht, hipStream_t s) {
  if (T == 0) return PQ_OK;
  pq_prof_scope prof(PQP_SWIGLU, s);
  const int per_lane = (F / 8 + 63) / 64;
  dim3 grid((T + 3) / 4), block(256);
  const uint16_t* u = (const uint16_t*)U;
  const uint16_t* g = (const uint16_t*)G;
  if (per_lane <= 4) swiglu_quant_kernel<4><<<grid, block, 0, s>>>(u, g, T, F, Fv, Hq, gamma, (uint16_t*)Ht);
  else if (per_lane <= 12) swiglu_quant_kernel<12><<<grid, block, 0, s>>>(u, g, T, F, Fv, Hq, gamma, (uint16_t*)Ht);
  else swiglu_quant_kernel<0><<<grid, block, 0, s>>>(u, g, T, F, Fv, Hq, gamma, (uint16_t*)Ht);
  PQ_CHECK_LAUNCH("swiglu_quant_kernel");
  return PQ_OK;
}

int pq_launch_swiglu_bwd(const void* dHd, const void* U, const void* G, int T, int F, int Fv, void* dU, void* dG, hipStream_t s) {
  const size_t n = (size_t)T * F;
  if (n == 0) return PQ_OK;
  pq_prof_scope prof(PQP_SWIGLU, s);
  const size_t nvec = n / 8;
  size_t blocks = (nvec + 511) / 512;                // two vectors per thread and pass
  if (blocks > 8192) blocks = 8192;
  swiglu_bwd_kernel<<<(unsigned)blocks, 256, 0, s>>>((const uint16_t*)dHd, (const uint16_t*)U, (const uint16_t*)G, nvec, F, Fv,
                                                    (uint16_t*)dU, (uint16_t*)dG);
  PQ_CHECK_LAUNCH("swiglu_bwd_kernel");
  return PQ_OK;
}

int pq_launch_expert_act(const void* ue, const void* ge, int ld, int S, int r, void* a, hipStream_t s) {
  const size_t n = (size_t)S * r;
  if (n == 0) return PQ_OK;
  pq_prof_scope prof(PQP_MOE_ELEMENTWISE, s);
  expert_act_kernel<<<(unsigned)((n / 8 + 255) / 256), 256, 0, s>>>((const uint16_t*)ue, (const uint16_t*)ge, ld, r, n / 8, (uint16_t*)a);
  PQ_CHECK_LAUNCH("expert_act_kernel");
  return PQ_OK;
}

int pq_launch_expert_act_bwd(const void* da, const void* ue, const void* ge, const void* a, const int* perm, const float* gate,
                             float alpha, int S, int r, int ld, void* du, void* dg, void* as, float* dWr, int n_wr, const pq_reduce_job* jobs,
                             hipStream_t s) {
  const int ride = dWr ? 2 + (n_wr + 255) / 256 : 0;
  if (S == 0 && ride == 0) return PQ_OK;
  pq_prof_scope prof(PQP_MOE_ELEMENTWISE, s);
  const size_t nvec = (size_t)S * r / 8;
  expert_act_bwd_kernel<<<(unsigned)((nvec + 255) / 256) + ride, 256, 0, s>>>((const uint16_t*)da, (const uint16_t*)ue, (const uint16_t*)ge,
                                                                      (const uint16_t*)a, perm, gate, alpha, r, ld, nvec, (uint16_t*)du,
                                                                      (uint16_t*)dg, (uint16_t*)as, ride, dWr, n_wr, jobs[0], jobs[1]);
  PQ_CHECK_LAUNCH("expert_act_bwd_kernel");
  return PQ_OK;
}

int pq_rowdot_blocks(int S) { return (S + 3) / 4; }
int pq_launch_slot_grad(const void* dY, const void* Ys, const int* perm, const float* gate, float alpha, bool scale, int k, int S, int d,
                        void* dst, float* rd, double* partial, hipStream_t s) {
  if (S == 0) return PQ_OK;
  pq_prof_scope prof(PQP_MOE_ELEMENTWISE, s);
  if (scale) slot_grad_kernel<true><<<(S + 3) / 4, 256, 0, s>>>((const uint16_t*)dY, (const uint16_t*)Ys, perm, gate, alpha, k, S, d, (uint16_t*)dst, rd, partial);
  else slot_grad_kernel<false><<<(S + 3) / 4, 256, 0, s>>>((const uint16_t*)dY, (const uint16_t*)Ys, perm, gate, alpha, k, S, d, (uint16_t*)dst, rd, partial);
  PQ_CHECK_LAUNCH("slot_grad_kernel");
  return PQ_OK;
}

int pq_launch_combine_fwd(void* Y, const void* Ys, const int* inv, const float* gate, float alpha, int T, int k, int d, hipStream_t s) {
  if (T == 0) return PQ_OK;
  pq_prof_scope prof(PQP_MOE_ELEMENTWISE, s);
  combine_fwd_kernel<<<(T + 3) / 4, 256, 0, s>>>((uint16_t*)Y, (const uint16_t*)Ys, inv, gate, alpha, T, k, d);
  PQ_CHECK_LAUNCH("combine_fwd_kernel");
  return PQ_OK;
}

size_t pq_dwr_scratch_bytes(int T, int d, int E) {
  const int c = dwr_chunk(T, d);
  return (size_t)((T + c - 1) / c) * E * d * sizeof(float);
}
int pq_launch_dwr(const float* rd, const int* inv, const int* idx, const float* probs, float alpha, int k, float* dlogit, const void* X, int T,
                  int d, int E, float* part, float* dWr, const pq_reduce_job* jobs, hipStream_t s) {
  pq_prof_scope prof(PQP_MOE_ELEMENTWISE, s);
  const int chunk = dwr_chunk(T, d), nchunks = (T + chunk - 1) / chunk;
  if (nchunks > 0) {
    dim3 grid((d + 255) / 256, nchunks);
    if (chunk == 32) dwr_partial_kernel<32><<<grid, 256, 0, s>>>(rd, inv, idx, probs, alpha, k, dlogit, (const uint16_t*)X, T, d, E, part);
    else dwr_partial_kernel<128><<<grid, 256, 0, s>>>(rd, inv, idx, probs, alpha, k, dlogit, (const uint16_t*)X, T, d, E, part);
    PQ_CHECK_LAUNCH("dwr_partial_kernel");
  }
  dwr_final_kernel<<<(E * d + 255) / 256 + 2, 256, 0, s>>>(part, nchunks, E * d, dWr, jobs[0], jobs[1]);
  PQ_CHECK_LAUNCH("dwr_final_kernel");
  return PQ_OK;
}

int pq_launch_combine_bwd(void* dX, const void* dXs, const int* inv, const float* dlogit, const void* Wr, int T, int k, int d, int E,
                          hipStream_t s) {
  if (T == 0) return PQ_OK;
  pq_prof_scope prof(PQP_MOE_ELEMENTWISE, s);
  const size_t wr_bytes = (size_t)E * d * 2;
  const int grid_l = (T + 4 * CB_TOK - 1) / (4 * CB_TOK);
  if (E <= 64 && k <= 2 && wr_bytes <= 64 * 1024 && d == 2048)
    combine_bwd_lds_kernel<4, 2><<<grid_l, 256, wr_bytes, s>>>((uint16_t*)dX, (const uint16_t*)dXs, inv, dlogit, (const uint16_t*)Wr, T, k, E);
  else if (E <= 64 && k <= 2 && wr_bytes <= 64 * 1024 && d == 4096)
    combine_bwd_lds_kernel<8, 2><<<grid_l, 256, wr_bytes, s>>>((uint16_t*)dX, (const uint16_t*)dXs, inv, dlogit, (const uint16_t*)Wr, T, k, E);
  else
    combine_bwd_kernel<<<(T + 3) / 4, 256, 0, s>>>((uint16_t*)dX, (const uint16_t*)dXs, inv, dlogit, (const uint16_t*)Wr, T, k, d, E);
  PQ_CHECK_LAUNCH("combine_bwd_kernel");
  return PQ_OK;
}
