// Pieces shared by the MFMA GEMM kernels (pq_gemm.hip, pq_tile.hip): the epilogue over eight consecutive columns and the
// expansion of packed signs into MFMA operands.
#pragma once
#include <string.h>
#include <type_traits>
#include "pq_internal.h"

typedef int pq_i32x2 __attribute__((ext_vector_type(2)));
#define PQ_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

namespace {

// The second problem of a paired launch as a kernel argument: empty in kernels that are never paired.
struct pq_no_second {};
template <bool PAIR>
using pq_second_arg = typename std::conditional<PAIR, pq_gemm_second, pq_no_second>::type;
template <bool PAIR>
pq_second_arg<PAIR> second_arg(const pq_gemm_second* second) {
  if constexpr (PAIR) {
    if (second) return *second;
    pq_gemm_second none;
    memset(&none, 0, sizeof(none));
    return none;
  } else return pq_no_second{};
}

// The derivative of the gated unit (Hd = silu(G) U) on eight columns, from the bf16 values: dU = dh silu(G), dG = dh U silu'(G); columns
// from Fv on do not exist and become zeros.
__device__ __forceinline__ void pq_swiglu_bwd8(const uint4& dh4, const uint4& u4, const uint4& g4, int col, int Fv, uint4& du4, uint4& dg4) {
  const uint32_t* d = &dh4.x;
  const uint32_t* u = &u4.x;
  const uint32_t* g = &g4.x;
  uint32_t* du = &du4.x;
  uint32_t* dg = &dg4.x;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    float o[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float dh = __uint_as_float(h ? d[w] & 0xFFFF0000u : d[w] << 16), uf = __uint_as_float(h ? u[w] & 0xFFFF0000u : u[w] << 16),
                  gf = __uint_as_float(h ? g[w] & 0xFFFF0000u : g[w] << 16);
      const float sg = pq_sigmoid(gf);
      const bool ok = col + 2 * w + h < Fv;
      o[0][h] = ok ? dh * (gf * sg) : 0.0f;
      o[1][h] = ok ? dh * uf * (sg * (1.0f + gf * (1.0f - sg))) : 0.0f;
    }
    du[w] = pack_bf16x2(o[0][0], o[0][1]);
    dg[w] = pack_bf16x2(o[1][0], o[1][1]);
  }
}

// ---------------------------------------------------------------------------------------------
// Epilogue
// ---------------------------------------------------------------------------------------------
struct epi_state {
  float sc0;
  float mu;
  double psum;
};

__device__ __forceinline__ void epi_begin(const pq_epilogue& e, epi_state& st) {
  st.sc0 = e.dev_scale ? __fmul_rn(e.scale, *e.dev_scale) : e.scale;
  st.mu = e.mu_dev ? *e.mu_dev : 0.0f;
  st.psum = 0.0;
}

__device__ __forceinline__ float load_io(const void* p, int kind, size_t i) {
  return kind == PQ_OUT_BF16 ? bf16_to_f32(((const uint16_t*)p)[i]) : ((const float*)p)[i];
}

template <int NT>
__device__ __forceinline__ void epi_end(const pq_epilogue& e, epi_state& st, double* red, int block_linear) {
  if (e.partials) {
    double t = block_sum_d<NT>(st.psum, red);
    if (threadIdx.x == 0) e.partials[block_linear] = t;
  }
}

// Eight consecutive columns of one output row (MFMA engine; widths and leading dimensions are
// multiples of 8, so every group is either fully inside or fully outside the matrix).
__device__ __forceinline__ void load_io8(const void* p, int kind, size_t i, float* f) {
  if (kind == PQ_OUT_BF16) {
    const uint4 u = *reinterpret_cast<const uint4*>((const uint16_t*)p + i);
    f[0] = __uint_as_float(u.x << 16); f[1] = __uint_as_float(u.x & 0xFFFF0000u);
    f[2] = __uint_as_float(u.y << 16); f[3] = __uint_as_float(u.y & 0xFFFF0000u);
    f[4] = __uint_as_float(u.z << 16); f[5] = __uint_as_float(u.z & 0xFFFF0000u);
    f[6] = __uint_as_float(u.w << 16); f[7] = __uint_as_float(u.w & 0xFFFF0000u);
  } else {
    const float4 a = *reinterpret_cast<const float4*>((const float*)p + i);
    const float4 b = *reinterpret_cast<const float4*>((const float*)p + i + 4);
    f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w; f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
  }
}

// row_scale: sc0 / row_div[m] when the caller has it at hand (NaN = not given, it is formed here).  TWO: the epilogue may have a
// second destination (C2, m_split); a template argument because the address arithmetic, inlined into every kernel, cost registers
// in all of them (step of 8192 tokens 2048x2048 r=128: 275.3 us with it everywhere, 272.1 without).
template <bool INT8, bool TWO = false>
__device__ __forceinline__ void epi_vec8(const pq_epilogue& e, epi_state& st, int m, int n, const uint4& r0,
                                         const uint4& r1, float row_scale = __builtin_nanf("")) {
  size_t ci = (size_t)m * e.ldc + n;
  if ((e.m_limit > 0 && m >= e.m_limit) || (e.n_limit > 0 && n >= e.n_limit)) return;
  void* cdst = e.C;
  if (TWO && e.m_split > 0) {                        // uniform
    const int z = m / (2 * e.m_split), mm = m - z * 2 * e.m_split;
    const bool hi = mm >= e.m_split;
    ci = (size_t)(z * e.m_split + (hi ? mm - e.m_split : mm)) * e.ldc + n;
    if (hi) cdst = e.C2;
  }
  const bool half = e.n_limit > 0 && n + 8 > e.n_limit;   // only the first four columns exist
  if (e.out_kind == PQ_OUT_I32) {
    *reinterpret_cast<uint4*>((int*)e.C + ci) = r0;
    if (!half) *reinterpret_cast<uint4*>((int*)e.C + ci + 4) = r1;
    return;
  }
  float acc[8];
  if constexpr (INT8) {
    acc[0] = (float)(int)r0.x; acc[1] = (float)(int)r0.y; acc[2] = (float)(int)r0.z; acc[3] = (float)(int)r0.w;
    acc[4] = (float)(int)r1.x; acc[5] = (float)(int)r1.y; acc[6] = (float)(int)r1.z; acc[7] = (float)(int)r1.w;
  } else {
    acc[0] = __uint_as_float(r0.x); acc[1] = __uint_as_float(r0.y); acc[2] = __uint_as_float(r0.z); acc[3] = __uint_as_float(r0.w);
    acc[4] = __uint_as_float(r1.x); acc[5] = __uint_as_float(r1.y); acc[6] = __uint_as_float(r1.z); acc[7] = __uint_as_float(r1.w);
  }
  if (e.dot_comp) {
    float c[8];
    load_io8(e.dot_comp, e.comp_kind, (size_t)m * e.ld_comp + n, c);
#pragma unroll
    for (int j = 0; j < 8; ++j) st.psum += (double)c[j] * (double)acc[j];
  }
  if (e.sign_bytes) {
    const uint32_t byte = e.sign_bytes[(size_t)m * e.ld_sign + (n >> 3)];
#pragma unroll
    for (int j = 0; j < 8; ++j) st.psum += ((byte >> j) & 1u) ? (double)acc[j] : -(double)acc[j];
  }
  float sc = st.sc0;
  if (e.row_div) sc = (row_scale == row_scale) ? row_scale : sc / e.row_div[m];
  float val[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) val[j] = __fmul_rn(sc, acc[j]);
  if (e.col_div) {
    const float4 c0 = *reinterpret_cast<const float4*>(e.col_div + n), c1 = *reinterpret_cast<const float4*>(e.col_div + n + 4);
    const float cd[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
#pragma unroll
    for (int j = 0; j < 8; ++j) val[j] = val[j] / cd[j];
  }
  if (e.maskW) {
    float w[8];
    load_io8(e.maskW, e.mask_kind, ci, w);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (fabs((double)w[j] - (double)st.mu) > (double)e.tau) val[j] = 0.0f;
  }
  if (TWO && INT8 && e.C2) {                         // uniform
    *reinterpret_cast<uint4*>((uint16_t*)e.C2 + ci) =
        make_uint4(pack_bf16x2(val[0], val[1]), pack_bf16x2(val[2], val[3]), pack_bf16x2(val[4], val[5]), pack_bf16x2(val[6], val[7]));
#pragma unroll
    for (int j = 0; j < 8; ++j) val[j] = __fmul_rn(e.c2_scale, val[j]);
  }
  if (e.accumulate) {
    float c[8];
    load_io8(e.C, e.out_kind, ci, c);
#pragma unroll
    for (int j = 0; j < 8; ++j) val[j] += c[j];
  }
  if (e.out_kind == PQ_OUT_BF16) {
    if (half)
      *reinterpret_cast<uint2*>((uint16_t*)e.C + ci) = make_uint2(pack_bf16x2(val[0], val[1]), pack_bf16x2(val[2], val[3]));
    else
      *reinterpret_cast<uint4*>((uint16_t*)e.C + ci) =
          make_uint4(pack_bf16x2(val[0], val[1]), pack_bf16x2(val[2], val[3]), pack_bf16x2(val[4], val[5]),
                     pack_bf16x2(val[6], val[7]));
  } else {
    *reinterpret_cast<float4*>((float*)cdst + ci) = make_float4(val[0], val[1], val[2], val[3]);
    if (!half) *reinterpret_cast<float4*>((float*)cdst + ci + 4) = make_float4(val[4], val[5], val[6], val[7]);
  }
}

// MFMA operand of +/-1 values from packed bits (bit i set = +1, clear = -1, Eq. 4): 8 bits -> 8 bf16 (bits
// above the eighth are ignored), 16 bits -> 16 int8.
__device__ __forceinline__ i32x4_t pq_bits_to_bf16(uint32_t b) {
  const uint32_t nb = ~b;
  i32x4_t o;
#pragma unroll
  for (int d = 0; d < 4; ++d)
    o[d] = (int)(0x3F803F80u | ((nb << (15 - 2 * d)) & 0x00008000u) | ((nb << (30 - 2 * d)) & 0x80000000u));
  return o;
}
__device__ __forceinline__ i32x4_t pq_bits_to_i8(uint32_t b) {
  i32x4_t o;
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const uint32_t m = __umul24((b >> (4 * d)) & 0xFu, 0x00204081u) & 0x01010101u;
    o[d] = (int)__builtin_amdgcn_perm(0x000001FFu, 0x000001FFu, m);
  }
  return o;
}

}  // namespace
