// Device code of the sign packer (pq_quant.hip), for the launches of other files that it rides along with.
#pragma once
#include "pq_internal.h"

template <typename T> struct vec16;  // 16 bytes of T
template <> struct vec16<float> {
  static constexpr int V = 4;
  static __device__ __forceinline__ void unpack(const uint4& u, float* f) {
    f[0] = __uint_as_float(u.x); f[1] = __uint_as_float(u.y);
    f[2] = __uint_as_float(u.z); f[3] = __uint_as_float(u.w);
  }
};
template <> struct vec16<uint16_t> {
  static constexpr int V = 8;
  static __device__ __forceinline__ void unpack(const uint4& u, float* f) {
    f[0] = __uint_as_float(u.x << 16); f[1] = __uint_as_float(u.x & 0xFFFF0000u);
    f[2] = __uint_as_float(u.y << 16); f[3] = __uint_as_float(u.y & 0xFFFF0000u);
    f[4] = __uint_as_float(u.z << 16); f[5] = __uint_as_float(u.z & 0xFFFF0000u);
    f[6] = __uint_as_float(u.w << 16); f[7] = __uint_as_float(u.w & 0xFFFF0000u);
  }
};

// ------------------------------------------------------------------------------------------
// Stage 2 + binarise + pack.  A block owns a 32-row x 512-column tile of W: every lane turns 8
// consecutive weights into one byte of the row-packed stream (LSB = lowest column), the bytes
// also go to LDS, from which the column-packed orientation (32 rows per word) is assembled.
// ------------------------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ uint32_t sign_byte(const T* p, float mu);
template <>
__device__ __forceinline__ uint32_t sign_byte<uint16_t>(const uint16_t* p, float mu) {
  float f[8];
  vec16<uint16_t>::unpack(*reinterpret_cast<const uint4*>(p), f);
  uint32_t b = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) b |= (f[j] >= mu ? 1u : 0u) << j;
  return b;
}
template <>
__device__ __forceinline__ uint32_t sign_byte<float>(const float* p, float mu) {
  float f[8];
  vec16<float>::unpack(*reinterpret_cast<const uint4*>(p), f);
  vec16<float>::unpack(*reinterpret_cast<const uint4*>(p + 4), f + 4);
  uint32_t b = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) b |= (f[j] >= mu ? 1u : 0u) << j;
  return b;
}

// RAGGED: K is a multiple of 4 but not of 32, or N is not a multiple of 32 (Table 1: D_ff - r = 5076).  Rows may then start
// on 8-byte (bf16) boundaries only and end inside a lane's 8 weights, so the weights are fetched as two halves of four, each
// wholly inside or wholly outside its row; everything outside (columns K..Kp-1 of a packed row, Kp = K rounded up to whole
// words, and rows N.. of the last word of the transposed packing) is packed as +1: a padded position only ever meets an
// activation code (or gradient) of zero.
template <typename T, bool RAGGED>
__device__ __forceinline__ void pack_sign_body(const T* __restrict__ W, int N, int K, const double* __restrict__ partials, int G,
                                               uint8_t* __restrict__ Pbytes, uint32_t* __restrict__ Pt, float* __restrict__ mu_lambda,
                                               int bx, int by) {
  __shared__ double red[4];
  __shared__ float s_mu;
  __shared__ uint8_t tileb[32][64];
  // the weights do not depend on the statistics: their eight chunks are requested first, so that their latency and
  // the reduction of the partial sums overlap instead of standing in a row
  constexpr int NU = sizeof(T) == 2 ? 1 : 2;          // 16-byte loads per 8 weights
  const int Kp = (K + 31) & ~31;
  const int n0 = by * 32, k0 = bx * 512;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int k = k0 + lane * 8;
  uint4 wv[8][NU];
#pragma unroll
  for (int rr = 0; rr < 8; ++rr) {
    const int row = n0 + w * 8 + rr;
    if constexpr (RAGGED) {
      // halves of four weights: 8 bytes (bf16) or 16 bytes (fp32), aligned because K % 4 == 0
      const bool in0 = row < N && k + 4 <= K, in1 = row < N && k + 8 <= K;
      const T* p0 = W + (in0 ? (size_t)row * K + k : (size_t)0);
      const T* p1 = W + (in1 ? (size_t)row * K + k + 4 : (size_t)0);
      if constexpr (sizeof(T) == 2) {
        const uint2 a = *reinterpret_cast<const uint2*>(p0), b = *reinterpret_cast<const uint2*>(p1);
        wv[rr][0] = make_uint4(a.x, a.y, b.x, b.y);
      } else {
        wv[rr][0] = *reinterpret_cast<const uint4*>(p0);
        wv[rr][1] = *reinterpret_cast<const uint4*>(p1);
      }
    } else {
      const bool in = row < N && k < K;
      const uint4* src = reinterpret_cast<const uint4*>(W + (in ? (size_t)row * K + k : (size_t)0));   // element (0, 0) always exists
#pragma unroll
      for (int u = 0; u < NU; ++u) wv[rr][u] = src[u];
    }
  }
  double s = 0.0, a = 0.0;
  for (int i = threadIdx.x; i < G; i += 256) {
    s += partials[2 * i];
    a += partials[2 * i + 1];
  }
  double ts = block_sum_d<256>(s, red);
  double ta = block_sum_d<256>(a, red);
  if (threadIdx.x == 0) {
    const double cnt = (double)N * (double)K;
    float mu = (float)(ts / cnt);
    s_mu = mu;
    if (bx == 0 && by == 0) {
      mu_lambda[0] = mu;
      mu_lambda[1] = (float)(ta / cnt);
    }
  }
  __syncthreads();
  const float mu = s_mu;
  const size_t kb = (size_t)Kp / 8;
#pragma unroll
  for (int rr = 0; rr < 8; ++rr) {
    const int rl = w * 8 + rr, row = n0 + rl;
    uint32_t b = RAGGED ? 0xFFu : 0u;
    if (row < N && k < Kp) {
      b = sign_byte<T>(reinterpret_cast<const T*>(wv[rr]), mu);
      if constexpr (RAGGED) {
        if (k + 4 > K) b |= 0x0Fu;
        if (k + 8 > K) b |= 0xF0u;
      }
      Pbytes[(size_t)row * kb + (k >> 3)] = (uint8_t)b;
    }
    tileb[rl][lane] = (uint8_t)b;
  }
  if (Pt == nullptr) return;
  __syncthreads();
  const size_t nw = ((size_t)N + 31) / 32;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int kk = threadIdx.x + h * 256;
    if (k0 + kk < K) {
      uint32_t word = 0;
#pragma unroll
      for (int j = 0; j < 32; ++j) word |= (((uint32_t)tileb[j][kk >> 3] >> (kk & 7)) & 1u) << j;
      Pt[(size_t)(k0 + kk) * nw + by] = word;
    }
  }
}
