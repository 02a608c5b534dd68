// Reference-precision engine (fp32 I/O): products and sums in fp64 on the matrix pipe (v_mfma_f64_16x16x4_f64), for every
// GEMM of the linear whose operands are fp32 but these: the 1-bit product of the forward, exact in int8, and the contractions of dX and dW
// of large calls, which come as int32 sums of digit products (pq_fixed.hip) that the SUM forms below add up in fp64.
//
// What bounds it: the instruction itself, 64 cycles per 2048 flops and SIMD (78.6 TFLOP/s over the chip; the vendor's fp64
// product reaches 71.8 on 4096^3).  A wavefront needs so little operand data per instruction (two 8-byte values per lane and
// 64 cycles at worst) that LDS staging buys nothing: every wavefront fetches its own fragments from global memory into
// registers several steps ahead and converts them on use, with no barrier anywhere in the loop.  What matters instead is
// that all 1024 SIMDs have equal work, so the wavefront tile is 64x64, 32x32 or 16x16 by the size of the output, four
// wavefronts share a small tile's contraction where even that leaves SIMDs idle, and independent products go into one launch.
// Accumulators stay in architectural registers (two wavefronts per SIMD in the launch bounds): with more than 256 registers
// allowed the compiler keeps them in AGPRs between the MFMAs and copies all of them out and back once per loop trip, which
// cost a quarter of the loop (an MFMA-only loop: 33 against 69 TFLOP/s).
// Measured against the LDS-staged 128x128 / 64x64 kernel that this replaced, one launch per product: 2048 tokens, 2048x2048,
// rank 128, forward and backward 2602 -> 724 us (dW 804 -> 275 us, dX with its rank-128 product 607 -> 277 us, i.e. 62 and 66
// TFLOP/s; H 251 -> 23 us); 64 tokens, 256x256, rank 16: 176 -> 37 us (13 -> 7 launches; 26 us in the 5 that are left).
#include <string.h>
#include "pq_epilogue.h"
#include "pq_pack.h"

namespace {

typedef double f64x4_t __attribute__((ext_vector_type(4)));

// A contraction step is 16 indices.  The assignment of indices to MFMA positions is free as long as both operands agree:
// lane (li, lk) = (lane & 15, lane >> 4) holds indices 4 lk .. 4 lk + 3 of its rows, one per instruction, so a
// contraction-contiguous operand arrives as one 16-byte load per row.  Rows are interleaved: block b's row li is row
// NB li + b of the tile, so a contraction-strided operand arrives as one NB-element load per index, and a lane's NB output
// columns are neighbours in memory.
// A fragment's loads are a base pointer that is the same for the wavefront (it advances by whole steps) plus lane offsets
// fixed in setup(), so that a step costs no address arithmetic on the vector unit (64-bit products per load had cost more
// than the MFMAs they fed on 32x32 tiles).  Only the partial step at the end of a contraction clamps its indices.
template <int KIND, int NB>
struct ref_frag;
struct ref_src {            // one operand of one wavefront tile: where step 0 starts, bytes per step, bytes per index (strided kinds)
  const char* p;
  size_t step;
  const float* kdiv;
  long ld;
};

template <int NB>
struct ref_frag<PQ_SRC_KC32, NB> {                       // fp32 rows, contraction contiguous (contraction length % 4 == 0)
  float4 v[NB];
  static __device__ __forceinline__ ref_src source(const pq_operand& op, int row0) {
    return ref_src{(const char*)op.p + (size_t)row0 * op.ld * 4, 64, nullptr, op.ld};
  }
  static constexpr int NOFF = NB;
  static __device__ __forceinline__ void offsets(uint32_t (&off)[NOFF], const ref_src& s, int r, int rows, int lk) {
#pragma unroll
    for (int b = 0; b < NB; ++b) off[b] = (uint32_t)min(r + b, rows - 1) * (uint32_t)s.ld * 4u + (uint32_t)lk * 16u;
  }
  __device__ __forceinline__ void load(const ref_src& s, const uint32_t (&off)[NOFF], int step) {
    const char* base = s.p + (size_t)step * s.step;
#pragma unroll
    for (int b = 0; b < NB; ++b) v[b] = *reinterpret_cast<const float4*>(base + off[b]);
  }
  __device__ __forceinline__ void load_tail(const ref_src& s, const uint32_t (&off)[NOFF], int step, int left, int lk) {
    const char* base = s.p + (size_t)step * s.step;
#pragma unroll
    for (int b = 0; b < NB; ++b) {                       // lanes past the end read the step's first four indices and drop them
      const bool in = 4 * lk < left;
      const float4 t = *reinterpret_cast<const float4*>(base + (in ? off[b] : off[b] - (uint32_t)lk * 16u));
      v[b] = in ? t : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
  __device__ __forceinline__ void ready(int) {}
  __device__ __forceinline__ double get(int b, int kk) const { return (double)(kk == 0 ? v[b].x : kk == 1 ? v[b].y : kk == 2 ? v[b].z : v[b].w); }
};

// contraction-strided kinds: one load of NB elements per index
template <int NB, int ES>
struct ref_strided {
  static __device__ __forceinline__ ref_src source(const pq_operand& op, int row0) {
    return ref_src{(const char*)op.p + (size_t)row0 * ES, (size_t)16 * op.ld * ES, op.kdiv, op.ld};
  }
  static constexpr int NOFF = 4;
  static __device__ __forceinline__ void offsets(uint32_t (&off)[NOFF], const ref_src& s, int r, int rows, int lk) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) off[kk] = ((uint32_t)(4 * lk + kk) * (uint32_t)s.ld + (uint32_t)min(r, rows - NB)) * (uint32_t)ES;
  }
  // offset of an index past the end: the step's first index
  static __device__ __forceinline__ uint32_t clamped(const ref_src& s, uint32_t off, int k, int left) {
    return k < left ? off : off - (uint32_t)k * (uint32_t)s.ld * (uint32_t)ES;
  }
};

template <int NB>
struct ref_frag<PQ_SRC_KS32, NB> : ref_strided<NB, 4> {  // fp32 (row count % NB == 0)
  using base_t = ref_strided<NB, 4>;
  float v[4][NB];
  __device__ __forceinline__ void fetch(const char* p, int kk) {
    if constexpr (NB == 4) {
      const float4 t = *reinterpret_cast<const float4*>(p);
      v[kk][0] = t.x; v[kk][1] = t.y; v[kk][2] = t.z; v[kk][3] = t.w;
    } else if constexpr (NB == 2) {
      const float2 t = *reinterpret_cast<const float2*>(p);
      v[kk][0] = t.x; v[kk][1] = t.y;
    } else v[kk][0] = *reinterpret_cast<const float*>(p);
  }
  __device__ __forceinline__ void load(const ref_src& s, const uint32_t (&off)[4], int step) {
    const char* base = s.p + (size_t)step * s.step;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) fetch(base + off[kk], kk);
  }
  __device__ __forceinline__ void load_tail(const ref_src& s, const uint32_t (&off)[4], int step, int left, int lk) {
    const char* base = s.p + (size_t)step * s.step;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) fetch(base + base_t::clamped(s, off[kk], 4 * lk + kk, left), kk);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int b = 0; b < NB; ++b) v[kk][b] = 4 * lk + kk < left ? v[kk][b] : 0.f;
  }
  __device__ __forceinline__ void ready(int) {}
  __device__ __forceinline__ double get(int b, int kk) const { return (double)v[kk][b]; }
};

template <int NB>
struct ref_frag<PQ_SRC_KS8, NB> : ref_strided<NB, 1> {   // int8 codes, each divided by kdiv of its index
  using base_t = ref_strided<NB, 1>;
  uint32_t v[4];
  float g[4];
  double rg[4];
  __device__ __forceinline__ void fetch(const char* p, int kk) {
    if constexpr (NB == 4) v[kk] = *reinterpret_cast<const uint32_t*>(p);
    else if constexpr (NB == 2) v[kk] = *reinterpret_cast<const uint16_t*>(p);
    else v[kk] = *reinterpret_cast<const uint8_t*>(p);
  }
  __device__ __forceinline__ void load(const ref_src& s, const uint32_t (&off)[4], int step) {
    const char* base = s.p + (size_t)step * s.step;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) fetch(base + off[kk], kk);
    const float4 t = *reinterpret_cast<const float4*>(s.kdiv + (size_t)step * 16 + 4 * ((threadIdx.x & 63) >> 4));
    g[0] = t.x; g[1] = t.y; g[2] = t.z; g[3] = t.w;
  }
  __device__ __forceinline__ void load_tail(const ref_src& s, const uint32_t (&off)[4], int step, int left, int lk) {
    const char* base = s.p + (size_t)step * s.step;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      fetch(base + base_t::clamped(s, off[kk], 4 * lk + kk, left), kk);
      g[kk] = s.kdiv[(size_t)step * 16 + (4 * lk + kk < left ? 4 * lk + kk : 0)];
    }
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) v[kk] = 4 * lk + kk < left ? v[kk] : 0u;
  }
  // 1 / gamma in fp64, one per index: the hardware estimate refined twice by Newton's iteration (gamma = 128 / max is a
  // normal, positive number), then one product per element
  __device__ __forceinline__ void ready(int) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const double d = (double)g[kk];
      double r = __builtin_amdgcn_rcp(d);
      r = __builtin_fma(r, __builtin_fma(-d, r, 1.0), r);
      rg[kk] = __builtin_fma(r, __builtin_fma(-d, r, 1.0), r);
    }
  }
  __device__ __forceinline__ double get(int b, int kk) const { return (double)(int8_t)(v[kk] >> (8 * b)) * rg[kk]; }
};

template <int NB>
struct ref_frag<PQ_SRC_BITSF, NB> {                      // packed signs, set = +1 (contraction length % 32 == 0: no partial step)
  uint32_t v[NB];
  static __device__ __forceinline__ ref_src source(const pq_operand& op, int row0) {
    return ref_src{(const char*)op.p + (size_t)row0 * op.ld, 2, nullptr, op.ld};
  }
  static constexpr int NOFF = NB;
  static __device__ __forceinline__ void offsets(uint32_t (&off)[NOFF], const ref_src& s, int r, int rows, int) {
#pragma unroll
    for (int b = 0; b < NB; ++b) off[b] = (uint32_t)min(r + b, rows - 1) * (uint32_t)s.ld;
  }
  __device__ __forceinline__ void load(const ref_src& s, const uint32_t (&off)[NOFF], int step) {
    const char* base = s.p + (size_t)step * s.step;
#pragma unroll
    for (int b = 0; b < NB; ++b) v[b] = *reinterpret_cast<const uint16_t*>(base + off[b]);
  }
  __device__ __forceinline__ void load_tail(const ref_src& s, const uint32_t (&off)[NOFF], int step, int, int) { load(s, off, step); }
  uint32_t n[NB];
  __device__ __forceinline__ void ready(int lk) {        // this lane's four bits, inverted, from bit 0 on
#pragma unroll
    for (int b = 0; b < NB; ++b) n[b] = ~(v[b] >> (4 * lk));
  }
  __device__ __forceinline__ double get(int b, int kk) const {   // +-1.0: the sign goes straight into the high word
    return __builtin_bit_cast(double, (uint64_t)(((n[b] << (31 - kk)) & 0x80000000u) | 0x3FF00000u) << 32);
  }
};

template <int AK, int BK, int NB>
__device__ __forceinline__ void ref_multiply(ref_frag<AK, NB>& fa, ref_frag<BK, NB>& fb, int lk, f64x4_t (&acc)[NB][NB]) {
  fa.ready(lk);
  fb.ready(lk);
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    double a[NB], b[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) { a[i] = fa.get(i, kk); b[i] = fb.get(i, kk); }
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
  }
}

// The contraction of one wavefront: steps first, first + stride, ... of 16 indices.  DEPTH steps are in flight.
template <int AK, int BK, int NB, int DEPTH>
__device__ __forceinline__ void ref_contract(const pq_operand& A, const pq_operand& B, int m0, int M, int n0, int N, int K, int first,
                                             int stride, int li, int lk, f64x4_t (&acc)[NB][NB]) {
  using FA = ref_frag<AK, NB>;
  using FB = ref_frag<BK, NB>;
  const int full = K >> 4, left = K & 15;
  const ref_src sa = FA::source(A, m0), sb = FB::source(B, n0);
  uint32_t oa[FA::NOFF], ob[FB::NOFF];
  FA::offsets(oa, sa, NB * li, M - m0, lk);
  FB::offsets(ob, sb, NB * li, N - n0, lk);
  if (first < full) {                                    // uniform for the wavefront
    FA fa[DEPTH];
    FB fb[DEPTH];
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) {
      const int t = min(first + u * stride, full - 1);
      fa[u].load(sa, oa, t);
      fb[u].load(sb, ob, t);
    }
    for (int s0 = first; s0 < full; s0 += DEPTH * stride) {
#pragma unroll
      for (int u = 0; u < DEPTH; ++u) {
        const int s = s0 + u * stride;
        if (s < full) {                                  // uniform
          ref_multiply<AK, BK, NB>(fa[u], fb[u], lk, acc);
          const int t = min(s + DEPTH * stride, full - 1);   // past the end: the last step again, never used
          fa[u].load(sa, oa, t);
          fb[u].load(sb, ob, t);
        }
      }
    }
  }
  if (left && (full - first) % stride == 0 && full >= first) {   // uniform: the partial step belongs to this wavefront
    FA fa;
    FB fb;
    fa.load_tail(sa, oa, full, left, lk);
    fb.load_tail(sb, ob, full, left, lk);
    ref_multiply<AK, BK, NB>(fa, fb, lk, acc);
  }
}

// The sums of a SUM form (a lane's two columns of a row are one load).
// False for the whole wavefront when one of its rows has no digits, or (FORM SUM_SS8, see pq_fixed.hip) one of its sums may consist
// of elements that the digits hold too coarsely: the tile is then to be formed as the fp64 product it stands for.
template <int FORM>
__device__ __forceinline__ bool ref_sums(const pq_ref_problem& p, int m0, int n0, int li, int lk, f64x4_t (&acc)[2][2]) {
  constexpr int NB = 2;
  const int n = min(n0 + NB * li, p.N - NB);
  const int rm = min(m0 + ((int)threadIdx.x & 31), p.M - 1);
  bool leave = p.exps[rm] == PQ_FIXED_NOT_FINITE;
  if constexpr (FORM == PQ_REF_SUM_SS8) {
    const int small = p.counts[rm], l = p.K - small - p.counts[p.M + rm];
    int z = p.counts[2 * p.M + min(n0 + ((int)threadIdx.x & 31), p.N - 1)];
    z = z == p.K ? 0 : z;                            // (a channel of zeros has no sum; of the others the one with the most zeros decides)
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) z = max(z, __shfl_xor(z, o, 64));
    leave |= 8 * max(l - z, 0) < min(small, p.K - z);
  }
  if (__any(leave)) return false;
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int m = min(m0 + NB * (lk + 4 * v) + i, p.M - 1);
      const double2 t = *reinterpret_cast<const double2*>(p.sums + (size_t)m * p.N + n);
      acc[i][0][v] = t.x;
      acc[i][1][v] = t.y;
    }
  return true;
}

// One workgroup's tile of one product.  KS = 1: the four wavefronts own a 2 x 2 arrangement of tiles; KS = 4: they share one
// tile, wavefront w taking every fourth step, and wavefront 0 adds their sums in order.
template <int FORM, int NB, int KS>
__device__ __forceinline__ void ref_tile(const pq_ref_problem& p, int block, double* lds, double* red) {
  constexpr bool SUM = FORM == PQ_REF_SUM_CBITS || FORM == PQ_REF_SUM_SS8;
  constexpr int WT = 16 * NB, DEPTH = NB == 4 ? 2 : NB == 2 ? 3 : 4;
  static_assert(!SUM || (NB == 2 && KS == 1), "the SUM forms take 32x32 wavefront tiles");
  constexpr bool BITS = FORM == PQ_REF_CBITS || FORM == PQ_REF_SUM_CBITS, CODES = FORM == PQ_REF_SS8 || FORM == PQ_REF_SUM_SS8;
  constexpr int AK = (CODES || FORM == PQ_REF_SS) ? PQ_SRC_KS32 : PQ_SRC_KC32;
  constexpr int BK = FORM == PQ_REF_CC ? PQ_SRC_KC32 : BITS ? PQ_SRC_BITSF : CODES ? PQ_SRC_KS8 : PQ_SRC_KS32;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), li = lane & 15, lk = lane >> 4;
  const int nbn = (p.N + WT * (KS == 1 ? 2 : 1) - 1) / (WT * (KS == 1 ? 2 : 1));
  const int bm = block / nbn, bn = block % nbn;
  const int m0 = KS == 1 ? (2 * bm + (wave >> 1)) * WT : bm * WT, n0 = KS == 1 ? (2 * bn + (wave & 1)) * WT : bn * WT;
  f64x4_t acc[NB][NB];
  auto clear = [&] {
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[i][j] = f64x4_t{0.0, 0.0, 0.0, 0.0};
  };
  if constexpr (!SUM) clear();
  const int first = KS == 1 ? 0 : wave;
  const bool live = KS == 4 || (m0 < p.M && n0 < p.N);    // uniform for the wavefront
  if (live) {
    bool contract = true;                                 // uniform
    if constexpr (SUM) {
      contract = !ref_sums<FORM>(p, m0, n0, li, lk, acc);
      if (contract) clear();
    }
    if (contract) ref_contract<AK, BK, NB, DEPTH>(p.A, p.B, m0, p.M, n0, p.N, p.K, first, KS, li, lk, acc);
    if constexpr (BITS) {
      // the rank-r product rides in the same accumulators; the 1-bit sum carries its scale from here on
      const double sc1 = (double)(p.dev_scale1 ? __fmul_rn(p.scale1, *p.dev_scale1) : p.scale1);
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[i][j][v] *= sc1;
      if (p.K2 > 0) ref_contract<PQ_SRC_KC32, PQ_SRC_KS32, NB, DEPTH>(p.A2, p.B2, m0, p.M, n0, p.N, p.K2, first, KS, li, lk, acc);
    }
  }
  if constexpr (KS == 4) {
    constexpr int PER = NB * NB * 4;
    if (wave > 0) {
      double* dst = lds + ((size_t)(wave - 1) * PER) * 64 + lane;
#pragma unroll
      for (int e = 0; e < PER; ++e) dst[e * 64] = acc[e / (NB * 4)][(e / 4) % NB][e % 4];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        double t = acc[e / (NB * 4)][(e / 4) % NB][e % 4];
#pragma unroll
        for (int w = 0; w < 3; ++w) t += lds[((size_t)w * PER + e) * 64 + lane];
        acc[e / (NB * 4)][(e / 4) % NB][e % 4] = t;
      }
    }
  }
  // result layout: register v of lane (li, lk) is element (row lk + 4 v, column li) of a 16x16 block
  const pq_epilogue& e = p.epi;
  double psum = 0.0;
  if (live && (KS == 1 || wave == 0)) {
    const double sc = (double)(e.dev_scale ? __fmul_rn(e.scale, *e.dev_scale) : e.scale);
    const double mu = e.mu_dev ? (double)*e.mu_dev : 0.0;
    const int n = n0 + NB * li;
    // one extra matrix per product at most (C itself, the matrix of the dot product, or W for the clip mask): the
    // elements of two row blocks are requested before the first is used (clamped, no load under a branch of its own; all
    // four blocks at once would not fit the registers of a 64x64 tile)
    const float* ex = e.accumulate ? (const float*)e.C : e.dot_comp ? (const float*)e.dot_comp : (const float*)e.maskW;   // uniform
    const long ldx = e.dot_comp ? e.ld_comp : e.ldc;
    constexpr int IH = NB < 2 ? NB : 2;
#pragma unroll
    for (int ih = 0; ih < NB; ih += IH) {
    float x[IH][4][NB];
    if (ex) {
#pragma unroll
      for (int ii = 0; ii < IH; ++ii)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float* c = ex + (size_t)min(m0 + NB * (lk + 4 * v) + ih + ii, p.M - 1) * ldx + min(n, p.N - NB);
          if constexpr (NB == 4) {
            const float4 t = *reinterpret_cast<const float4*>(c);
            x[ii][v][0] = t.x; x[ii][v][1] = t.y; x[ii][v][2] = t.z; x[ii][v][3] = t.w;
          } else if constexpr (NB == 2) {
            const float2 t = *reinterpret_cast<const float2*>(c);
            x[ii][v][0] = t.x; x[ii][v][1] = t.y;
          } else x[ii][v][0] = *c;
        }
    }
#pragma unroll
    for (int ii = 0; ii < IH; ++ii)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = ih + ii;
        const int m = m0 + NB * (lk + 4 * v) + i;
        if (m >= p.M || n >= p.N) continue;
        if (e.dot_comp) {
#pragma unroll
          for (int j = 0; j < NB; ++j) psum += (double)x[ii][v][j] * acc[i][j][v];
        }
        if (e.sign_bytes) {                               // NB columns from column n (a multiple of NB): inside one byte
          const uint32_t bits = (uint32_t)e.sign_bytes[(size_t)m * e.ld_sign + (n >> 3)] >> (n & 7);
#pragma unroll
          for (int j = 0; j < NB; ++j) psum += ((bits >> j) & 1u) ? acc[i][j][v] : -acc[i][j][v];
        }
        float o[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          double val = sc * acc[i][j][v];
          if (e.maskW && fabs((double)x[ii][v][j] - mu) > (double)e.tau) val = 0.0;
          if (e.accumulate) val += (double)x[ii][v][j];
          o[j] = (float)val;
        }
        float* dst = (float*)e.C + (size_t)m * e.ldc + n;
        if constexpr (NB == 4) *reinterpret_cast<float4*>(dst) = make_float4(o[0], o[1], o[2], o[3]);
        else if constexpr (NB == 2) *reinterpret_cast<float2*>(dst) = make_float2(o[0], o[1]);
        else *dst = o[0];
      }
    }
  }
  if (e.partials) {                                       // uniform
    const double t = block_sum_d<256>(psum, red);
    if (threadIdx.x == 0) e.partials[block] = t;
  }
}

struct ref_launch {
  pq_ref_problem p[PQ_REF_MAX];
  int first[PQ_REF_MAX];                                  // first workgroup of each product
  int n, total;                                           // products; their workgroups (the reductions follow)
  pq_reduce_job jobs[2];
};

// BIG: 64x64 wavefront tiles (one wavefront per SIMD, 128 accumulator registers); otherwise the three small forms.
template <bool BIG>
__global__ __launch_bounds__(256, 2) void ref_gemm_kernel(ref_launch L) {
  __shared__ double red[4];
  const int b = blockIdx.x;
  if (b >= L.total) {                                     // uniform: the scalar reductions that ride along
    pq_reduce_job_body(b == L.total ? L.jobs[0] : L.jobs[1]);
    return;
  }
  // (selected with constant indices: a run-time index would move the argument block to scratch memory)
  pq_ref_problem p = L.p[0];
  int blk = b;
#pragma unroll
  for (int q = 1; q < PQ_REF_MAX; ++q)
    if (q < L.n && b >= L.first[q]) { p = L.p[q]; blk = b - L.first[q]; }
#define PQ_REF_FORMS(NB, KS, LDS)                                                     \
  switch (p.form) {                                                                   \
    case PQ_REF_CC: ref_tile<PQ_REF_CC, NB, KS>(p, blk, LDS, red); break;              \
    case PQ_REF_CS: ref_tile<PQ_REF_CS, NB, KS>(p, blk, LDS, red); break;              \
    case PQ_REF_CBITS: ref_tile<PQ_REF_CBITS, NB, KS>(p, blk, LDS, red); break;          \
    case PQ_REF_SS8: ref_tile<PQ_REF_SS8, NB, KS>(p, blk, LDS, red); break;        \
    default: ref_tile<PQ_REF_SS, NB, KS>(p, blk, LDS, red);                            \
  }
  if constexpr (BIG) {
    PQ_REF_FORMS(4, 1, nullptr)
  } else {
    __shared__ double lds[3 * 16 * 64];
    if (p.cfg == 1) {
      if (p.form == PQ_REF_SUM_CBITS) ref_tile<PQ_REF_SUM_CBITS, 2, 1>(p, blk, nullptr, red);   // (the SUM forms: always this one)
      else if (p.form == PQ_REF_SUM_SS8) ref_tile<PQ_REF_SUM_SS8, 2, 1>(p, blk, nullptr, red);
      else { PQ_REF_FORMS(2, 1, nullptr) }
    }
    else if (p.cfg == 2) { PQ_REF_FORMS(2, 4, lds) }
    else { PQ_REF_FORMS(1, 4, lds) }
  }
#undef PQ_REF_FORMS
}

// One product of the small forms beside the packing of an fp32 weight: the first `nref` workgroups are the product's.
// H = X A^T and the packing have no data in common and each leaves most CUs idle or waiting: forward and backward of 64 tokens, 256x256,
// r = 16 34.9 -> 31.6 us, 2048 tokens, 2048x2048, r = 128 377 -> 371 us.
struct ref_pack_args {
  pq_ref_problem p;
  const float* W;
  const double* partials;
  uint8_t* P;
  uint32_t* Pt;
  float* mu_lambda;
  int N, K, nparts, nref, gx;
};
template <bool RAGGED>
__global__ __launch_bounds__(256, 2) void ref_pack_kernel(ref_pack_args a) {
  const int b = blockIdx.x;
  if (b >= a.nref) {                                      // uniform
    const int t = b - a.nref;
    pack_sign_body<float, RAGGED>(a.W, a.N, a.K, a.partials, a.nparts, a.P, a.Pt, a.mu_lambda, t % a.gx, t / a.gx);
    return;
  }
  __shared__ double red[4];
  __shared__ double lds[3 * 16 * 64];
  if (a.p.cfg == 1) ref_tile<PQ_REF_CC, 2, 1>(a.p, b, nullptr, red);
  else if (a.p.cfg == 2) ref_tile<PQ_REF_CC, 2, 4>(a.p, b, lds, red);
  else ref_tile<PQ_REF_CC, 1, 4>(a.p, b, lds, red);
}

// Y = fl32(fl32(fl32(beta lambda) / gamma_t) * acc) + alpha H B^T of the fp32 forward in one launch: acc is the exact int8
// product of the codes with the packed signs, the rank-r product runs in fp64 and the sum is rounded once.  A workgroup owns
// 16 x 16 outputs, its wavefronts take every fourth step of both contractions.
// Bound by the latency of one chain of loads and by the launch itself (64 tokens, 256x256: 64 workgroups), so it is one launch of
// small workgroups where the int8 product and the fp64 product were one each.
// A 16x16 MFMA leaves rows 4 lk .. 4 lk + 3 in a lane in its int8 form and rows lk, lk + 4, .. in its fp64 form: the codes'
// rows are fed permuted, so that both sums of an output meet in one register.
__global__ __launch_bounds__(256) void ref_linear_kernel(pq_ref_linear p) {
  __shared__ int li8[3][4][64];
  __shared__ double lf64[3][4][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), li = lane & 15, lk = lane >> 4;
  const int nbn = (p.N + 15) / 16, m0 = (int)blockIdx.x / nbn * 16, n0 = (int)blockIdx.x % nbn * 16;
  const int n = n0 + li;
  i32x4_t acc = {0, 0, 0, 0};
  {
    const int8_t* qrow = p.Xq + (size_t)min(m0 + (li >> 2) + 4 * (li & 3), p.T - 1) * p.K;
    const uint8_t* prow = (const uint8_t*)p.P + (size_t)min(n, p.N - 1) * (p.K / 8);
    constexpr int D = 4;                                  // steps of 64 indices in flight; K is a multiple of 32: past it, index 0 and no codes
    for (int s0 = wave; s0 * 64 < p.K; s0 += 4 * D) {     // uniform
      i32x4_t a[D];
      uint32_t b[D];
#pragma unroll
      for (int u = 0; u < D; ++u) {
        const int k = (s0 + 4 * u) * 64 + 16 * lk;
        const bool in = k < p.K;
        const i32x4_t t = *reinterpret_cast<const i32x4_t*>(qrow + (in ? k : 0));
        a[u] = in ? t : i32x4_t{0, 0, 0, 0};
        b[u] = *reinterpret_cast<const uint16_t*>(prow + (in ? k >> 3 : 0));
      }
#pragma unroll
      for (int u = 0; u < D; ++u) acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[u], pq_bits_to_i8(b[u]), acc, 0, 0, 0);
    }
  }
  f64x4_t hb[1][1] = {{f64x4_t{0.0, 0.0, 0.0, 0.0}}};
  ref_contract<PQ_SRC_KC32, PQ_SRC_KC32, 1, 4>(p.H, p.B, m0, p.T, n0, p.N, p.r, wave, 4, li, lk, hb);
  if (wave > 0) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      li8[wave - 1][v][lane] = acc[v];
      lf64[wave - 1][v][lane] = hb[0][0][v];
    }
  }
  __syncthreads();
  if (wave > 0 || n >= p.N) return;
  const float sc1 = __fmul_rn(p.beta, *p.lambda);
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int m = m0 + lk + 4 * v;
    if (m >= p.T) continue;
    int t = acc[v];
    double h = hb[0][0][v];
#pragma unroll
    for (int w = 0; w < 3; ++w) {
      t += li8[w][v][lane];
      h += lf64[w][v][lane];
    }
    const float y = __fmul_rn(sc1 / p.gamma[m], (float)t);
    p.Y[(size_t)m * p.N + n] = (float)((double)p.alpha * h + (double)y);
  }
}

constexpr int kNB[4] = {4, 2, 2, 1}, kKS[4] = {1, 1, 4, 4};

int ref_blocks(int cfg, int M, int N) {
  const int t = 16 * kNB[cfg] * (kKS[cfg] == 1 ? 2 : 1);
  return ((M + t - 1) / t) * ((N + t - 1) / t);
}

// Wavefront tile and sharing of one product: the form whose busiest SIMD has the least to do, in MFMA instructions (each of
// the 1024 SIMDs gets every 1024th wavefront), weighted by what a form loses to its own loads and conversions: all products
// of 2048 tokens, 2048x2048, rank 128 forced into one form took 592 us (dW + dX, 64x64), 762 (32x32), 680 (32x32, shared
// contraction) and 1137 (16x16), while H (2048 x 128) took 252, 66, 24 and 35 us in the same order.
int ref_config(int M, int N, int K) {
  int best = 0;
  double cost = 0.0;
  const double lose[4] = {1.0, 1.35, 1.2, 2.0};
  for (int c = 0; c < 4; ++c) {
    const long waves = (long)ref_blocks(c, M, N) * 4;
    const long rounds = (waves + 1023) / 1024, steps = ((K + 15) / 16 + kKS[c] - 1) / kKS[c];
    const double t = (double)rounds * kNB[c] * kNB[c] * 4.0 * (double)(steps + 2) * lose[c];
    if (c == 0 || t < cost) { best = c; cost = t; }
  }
  return best;
}

}  // namespace

// (the SUM forms read a sum each: 32x32 tiles, in the launch of the small products)
int pq_ref_red_blocks(int M, int N, int K) { return ref_blocks(K < 0 ? 1 : ref_config(M, N, K), M, N); }

int pq_launch_ref(pq_ref_problem* p, int n, const pq_reduce_job* jobs, int njobs, hipStream_t s, int prof_label) {
  for (int i = 0; i < n; ++i)
    if ((p[i].epi.accumulate != 0) + (p[i].epi.dot_comp != nullptr) + (p[i].epi.maskW != nullptr) > 1)
      return pq_set_error(PQ_ERR_BAD_ARG, "reference engine: one extra matrix per product");
  if (n < 0 || n > PQ_REF_MAX || njobs < 0 || njobs > 2) return pq_set_error(PQ_ERR_BAD_ARG, "reference engine: %d products, %d reductions", n, njobs);
  bool jobs_left = njobs > 0, had_big = false;
  for (int big = 1; big >= 0; --big) {                    // 64x64 tiles first (they take longest)
    ref_launch L;
    memset(&L, 0, sizeof(L));
    int total = 0;
    for (int i = 0; i < n; ++i) {
      if (p[i].M <= 0 || p[i].N <= 0) continue;
      p[i].cfg = p[i].form == PQ_REF_SUM_CBITS || p[i].form == PQ_REF_SUM_SS8 ? 1 : ref_config(p[i].M, p[i].N, p[i].K);
      if ((p[i].cfg == 0) != (big == 1)) continue;
      L.p[L.n] = p[i];
      L.first[L.n++] = total;
      total += ref_blocks(p[i].cfg, p[i].M, p[i].N);
    }
    L.total = total;
    const bool with_jobs = jobs_left && (total > 0 || big == 0);
    if (with_jobs) {
      for (int j = 0; j < njobs; ++j) L.jobs[j] = jobs[j];
      total += njobs;
      jobs_left = false;
    }
    if (total == 0) continue;
    pq_prof_scope prof(big == 0 && had_big ? (int)PQP_GEMM_OTHER : prof_label, s);
    had_big = big == 1;
    if (big) ref_gemm_kernel<true><<<total, 256, 0, s>>>(L);
    else ref_gemm_kernel<false><<<total, 256, 0, s>>>(L);
    PQ_CHECK_LAUNCH("ref_gemm_kernel");
  }
  return PQ_OK;
}

// The product rides along with the packing when it takes one of the small forms.
bool pq_ref_rides(int M, int N, int K) { return M > 0 && N > 0 && ref_config(M, N, K) != 0; }

int pq_launch_ref_pack(const pq_ref_problem& p, const float* W, int N, int K, const double* partials, int nparts, uint32_t* P, uint32_t* Pt,
                       float* mu_lambda, hipStream_t s) {
  if (p.form != PQ_REF_CC || !pq_ref_rides(p.M, p.N, p.K)) return pq_set_error(PQ_ERR_BAD_ARG, "reference engine: product cannot ride along");
  pq_prof_scope prof(PQP_PACK, s);
  ref_pack_args a{p, W, partials, (uint8_t*)P, Pt, mu_lambda, N, K, nparts, 0, (((K + 31) & ~31) + 511) / 512};
  a.p.cfg = ref_config(p.M, p.N, p.K);
  a.nref = ref_blocks(a.p.cfg, p.M, p.N);
  const int blocks = a.nref + a.gx * ((N + 31) / 32);
  if (K % 32 != 0 || N % 32 != 0) ref_pack_kernel<true><<<blocks, 256, 0, s>>>(a);
  else ref_pack_kernel<false><<<blocks, 256, 0, s>>>(a);
  PQ_CHECK_LAUNCH("ref_pack_kernel");
  return PQ_OK;
}

// One resident round of 16x16 tiles (four workgroups on each of 256 CUs): below it the launch that goes is worth more than what
// larger tiles save, beyond it the two launches' 64x64 and 32x32 tiles are faster; contractions beyond 4096 gain nothing either way.
// Forward and backward, two launches against one: 64 tokens, 256x256, r = 16: 31.1 -> 26.1 us; 512 tokens (1024 tiles), 512x512, r = 64:
// 54.0 -> 52.6; 512 tokens, 4096x512: 150.7 -> 150.6; 256 tokens, 8192x1024: 286 -> 289; 2048 tokens (2048 tiles), 256x256, r = 256: 83 -> 90;
// 300 tokens (2432 tiles), 2048x2048: 162 -> 174.
bool pq_ref_linear_applies(int T, int N, int K) { return (long)((T + 15) / 16) * ((N + 15) / 16) <= 1024 && K <= 4096; }

int pq_launch_ref_linear(const pq_ref_linear& p, hipStream_t s) {
  if (p.K % 32 != 0 || p.r % 4 != 0) return pq_set_error(PQ_ERR_SHAPE, "K=%d must be a multiple of 32, r=%d of 4", p.K, p.r);
  pq_prof_scope prof(PQP_GEMM_ONEBIT, s);
  ref_linear_kernel<<<((p.T + 15) / 16) * ((p.N + 15) / 16), 256, 0, s>>>(p);
  PQ_CHECK_LAUNCH("ref_linear_kernel");
  return PQ_OK;
}
