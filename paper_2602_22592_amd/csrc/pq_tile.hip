// Streaming tile GEMM for gfx950: 64x64 and 128x128 output tiles on four wavefronts.
//
//   C[m][n] (+)= epilogue( sum_k A(m,k) * B(n,k) [then + sum_k2 A2(m,k2) * B2(n,k2)] )
//
// Takes what the 256x256 kernels of pq_gemm.hip leave idle: outputs of few tiles, narrow outputs, expert segments and
// contractions that are not whole steps.  Such a product is a chain of memory latencies, so everything here is about
// having the whole of it in flight: operand tiles of a 128-byte contraction step go from global memory straight into a
// ring of LDS stages.  128x128: NST stages, NST - 1 of them ahead of the MFMAs, one barrier per step, two workgroups per CU.
// 64x64: groups of two steps, one barrier per group; two groups (two workgroups per CU), or four while the launch leaves a
// workgroup a CU to itself; the second contraction's first tiles are requested before the first one's.
// A chunk past the end of the contraction is fetched from a page of zeros, so any length that is a whole number of 16-byte
// chunks (KC kinds) or of rows (KS16) runs without masks; rows and columns past the edge re-read a valid one and are not
// stored.  Packed signs stay packed in LDS (one dword per lane and load, no alignment beyond the word) and are expanded
// next to the MFMAs; past the end of a row they repeat its last word, where A is zero.
// LDS layouts: KC: [row][128 B], 16-byte chunk c at c ^ row ^ (row >> 3); KS16: [64 contraction rows][2 * TILE B] as it
// lies in memory, chunk c of row t at c ^ (TILE / 32) * (t & 3), read back with the transposing LDS read; signs: [row][16 or 8 B].
#include <string.h>
#include <type_traits>
#include "pq_epilogue.h"

namespace {

[[maybe_unused]] __device__ __attribute__((aligned(256))) unsigned char pq_zero_page[256];   // never written

// operand kinds that launches of two products come in: U and G, dW_up and dW_gate, dB and dA
template <int AK, int BK, int BK2>
constexpr bool pair_kinds() { return BK2 < 0 && ((AK == PQ_SRC_KS16 && BK == PQ_SRC_KS16) || (AK == PQ_SRC_KC8 && BK == PQ_SRC_BITS8)); }

// Operand tile of ROWS rows (or columns, KS16) x 128 bytes of contraction per step.
template <int KIND, int ROWS>
struct tile_src {
  static constexpr bool kStrided = KIND == PQ_SRC_KS16;
  static constexpr bool kBits = KIND == PQ_SRC_BITS8 || KIND == PQ_SRC_BITS16;
  static constexpr int ES = (KIND == PQ_SRC_KC8) ? 1 : 2;
  static constexpr int WPS = KIND == PQ_SRC_BITS8 ? 4 : 2;                       // bits: words per row and step
  static constexpr int BYTES = kBits ? ROWS * WPS * 4 : ROWS * 128;              // LDS bytes of a stage
  static constexpr int NBLK = kBits ? (ROWS * WPS + 63) / 64 : ROWS / 8;         // load instructions per stage
  static constexpr int LPW = NBLK >= 4 ? NBLK / 4 : 1;                           // ... per wavefront (fewer than four: repeated)
  static_assert(NBLK % 4 == 0 || 4 % NBLK == 0, "even split over the wavefronts");
  const char* src[LPW];
  int pos[LPW];          // KC: byte offset inside a step; KS16: contraction row inside a step; bits: word inside a step
  size_t adv;            // source bytes per step

  __device__ __forceinline__ static int blk(int wv, int i) { return NBLK >= 4 ? wv * LPW + i : wv % NBLK; }
  // kb: first contraction index of the range
  __device__ __forceinline__ void setup(const pq_operand& op, int row0, int rows, int kb, int wv, int lane) {
    adv = kStrided ? (size_t)64 * op.ld * 2 : kBits ? (size_t)WPS * 4 : (size_t)128;
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
      const int b = blk(wv, i);
      if constexpr (kStrided) {
        constexpr int CPR = ROWS / 8, TPB = 64 / CPR;                            // chunks per row, rows per block
        const int t = b * TPB + lane / CPR, pc = lane % CPR;
        int col = row0 + (pc ^ ((ROWS / 32) * (t & 3))) * 8;
        if (col + 8 > rows) col = row0;
        pos[i] = t;
        src[i] = (const char*)op.p + ((size_t)(kb + t) * op.ld + col) * 2;
      } else if constexpr (kBits) {
        const int r = b * (64 / WPS) + lane / WPS;
        pos[i] = lane % WPS;
        src[i] = (const char*)op.p + (size_t)min(row0 + r, rows - 1) * op.ld + (kb >> 3) + pos[i] * 4;
      } else {
        const int r = b * 8 + (lane >> 3);
        const int c = (lane & 7) ^ ((r ^ (r >> 3)) & 7);
        pos[i] = c * 16;
        src[i] = (const char*)op.p + ((size_t)min(row0 + r, rows - 1) * op.ld + kb) * ES + c * 16;
      }
    }
  }
  // step kt into the stage at `base`; klen: contraction indices of the range
  __device__ __forceinline__ void issue(int kt, int klen, unsigned char* base, int wv) const {
#if defined(__HIP_DEVICE_COMPILE__)
    const int step = (kStrided || KIND == PQ_SRC_KC16 || KIND == PQ_SRC_BITS16) ? 64 : 128;
    const bool whole = (kt + 1) * step <= klen;      // uniform
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
      const char* g = src[i] + (size_t)kt * adv;
      if (!whole) {
        if constexpr (kStrided) { if (kt * 64 + pos[i] >= klen) g = (const char*)pq_zero_page; }
        else if constexpr (kBits) { const int over = kt * WPS + pos[i] - ((klen >> 5) - 1); if (over > 0) g -= (size_t)over * 4; }
        else { if (kt * 128 + pos[i] >= klen * ES) g = (const char*)pq_zero_page; }
      }
      if constexpr (kBits) __builtin_amdgcn_global_load_lds(g, PQ_LDS_PTR(base + blk(wv, i) * 256), 4, 0, 0);
      else __builtin_amdgcn_global_load_lds(g, PQ_LDS_PTR(base + blk(wv, i) * 1024), 16, 0, 0);
    }
#endif
  }
};

// Fragment addresses (stage 0) of the NB 32-row blocks of an operand that a wavefront owns.
template <int KIND, int ROWS, int NB>
struct tile_frag {
  uint32_t ad[NB];
  __device__ __forceinline__ void setup(uint32_t lds0, int w0, int lane) {
    const int h = lane >> 5;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int r = w0 + 32 * j + (lane & 31);
      if constexpr (KIND == PQ_SRC_KS16) {
        const int t = 8 * h + ((lane & 15) >> 2), col = w0 + 32 * j + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
        ad[j] = lds0 + t * (ROWS * 2) + (((col >> 3) ^ ((ROWS / 32) * (t & 3))) << 4) + (col & 7) * 2;
      } else if constexpr (KIND == PQ_SRC_BITS8 || KIND == PQ_SRC_BITS16) ad[j] = lds0 + r * (KIND == PQ_SRC_BITS8 ? 16 : 8);
      else ad[j] = lds0 + r * 128 + (((h ^ r ^ (r >> 3)) & 7) << 4);   // sub-step ks: address ^ (ks << 5)
    }
  }
};

// LDS reads are asm blocks that carry their own wait, so a register is valid when its block ends; what a wavefront needs
// next goes into one block: two sub-steps of a 128x128 step (all four with packed signs).  (Reads per sub-step with a wait
// each ran a 64x64 step in 1000 clocks whatever the depth of the ring.)  t, u: 8-byte halves of transposing reads, two per operand.
__device__ __forceinline__ i32x4_t join(const pq_i32x2& lo, const pq_i32x2& hi) { return i32x4_t{lo[0], lo[1], hi[0], hi[1]}; }
#define RD "ds_read_b128 "
#define RT "ds_read_b64_tr_b16 "
#define W0 "s_waitcnt lgkmcnt(0)"

// Two 32-row blocks per operand (128x128 tiles), sub-steps ks and ks + 1 (x = ks << 5): o[2 * (ks & 1) + block].
__device__ __forceinline__ void rd_kc_kc_x2(i32x4_t* a, i32x4_t* b, uint32_t p0, uint32_t p1, uint32_t r0, uint32_t r1, uint32_t x) {
  asm volatile(RD "%0, %8\n\t" RD "%4, %12\n\t" RD "%1, %9\n\t" RD "%5, %13\n\t" RD "%2, %10\n\t" RD "%6, %14\n\t" RD "%3, %11\n\t" RD "%7, %15\n\t" W0
               : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3]), "=&v"(b[0]), "=&v"(b[1]), "=&v"(b[2]), "=&v"(b[3])
               : "v"(p0 ^ x), "v"(p1 ^ x), "v"(p0 ^ (x + 32u)), "v"(p1 ^ (x + 32u)), "v"(r0 ^ x), "v"(r1 ^ x), "v"(r0 ^ (x + 32u)), "v"(r1 ^ (x + 32u))
               : "memory");
}
template <int R>   // R: bytes of a contraction row of the KS16 tile; r0, r1 already at the first sub-step's rows
__device__ __forceinline__ void rd_kc_ks_x2(i32x4_t* a, i32x4_t* b, uint32_t p0, uint32_t p1, uint32_t r0, uint32_t r1, uint32_t x) {
  pq_i32x2 t[8];
  asm volatile(RD "%0, %12\n\t" RT "%4, %16\n\t" RT "%5, %16 offset:%18\n\t" RD "%1, %13\n\t" RT "%6, %17\n\t" RT "%7, %17 offset:%18\n\t"
               RD "%2, %14\n\t" RT "%8, %16 offset:%19\n\t" RT "%9, %16 offset:%20\n\t" RD "%3, %15\n\t" RT "%10, %17 offset:%19\n\t" RT "%11, %17 offset:%20\n\t" W0
               : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3]), "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3]), "=&v"(t[4]), "=&v"(t[5]),
                 "=&v"(t[6]), "=&v"(t[7])
               : "v"(p0 ^ x), "v"(p1 ^ x), "v"(p0 ^ (x + 32u)), "v"(p1 ^ (x + 32u)), "v"(r0), "v"(r1), "n"(4 * R), "n"(16 * R), "n"(20 * R) : "memory");
#pragma unroll
  for (int k = 0; k < 4; ++k) b[k] = join(t[2 * k], t[2 * k + 1]);
}
template <int R>
__device__ __forceinline__ void rd_ks_ks_x2(i32x4_t* a, i32x4_t* b, uint32_t p0, uint32_t p1, uint32_t r0, uint32_t r1) {
  pq_i32x2 t[8], u[8];
  asm volatile(RT "%0, %16\n\t" RT "%1, %16 offset:%20\n\t" RT "%8, %18\n\t" RT "%9, %18 offset:%20\n\t"
               RT "%2, %17\n\t" RT "%3, %17 offset:%20\n\t" RT "%10, %19\n\t" RT "%11, %19 offset:%20\n\t"
               RT "%4, %16 offset:%21\n\t" RT "%5, %16 offset:%22\n\t" RT "%12, %18 offset:%21\n\t" RT "%13, %18 offset:%22\n\t"
               RT "%6, %17 offset:%21\n\t" RT "%7, %17 offset:%22\n\t" RT "%14, %19 offset:%21\n\t" RT "%15, %19 offset:%22\n\t" W0
               : "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3]), "=&v"(t[4]), "=&v"(t[5]), "=&v"(t[6]), "=&v"(t[7]),
                 "=&v"(u[0]), "=&v"(u[1]), "=&v"(u[2]), "=&v"(u[3]), "=&v"(u[4]), "=&v"(u[5]), "=&v"(u[6]), "=&v"(u[7])
               : "v"(p0), "v"(p1), "v"(r0), "v"(r1), "n"(4 * R), "n"(16 * R), "n"(20 * R) : "memory");
#pragma unroll
  for (int k = 0; k < 4; ++k) { a[k] = join(t[2 * k], t[2 * k + 1]); b[k] = join(u[2 * k], u[2 * k + 1]); }
}
// both blocks of A for all four sub-steps (o[2 * ks + block]) and the packed words of both B blocks
template <bool WIDE>
__device__ __forceinline__ void rd_kc_bits_x4(i32x4_t* o, i32x4_t* q, uint32_t p0, uint32_t p1, uint32_t r0, uint32_t r1) {
  if constexpr (WIDE)
    asm volatile(RD "%8, %18\n\t" RD "%9, %19\n\t" RD "%0, %10\n\t" RD "%1, %14\n\t" RD "%2, %11\n\t" RD "%3, %15\n\t" RD "%4, %12\n\t" RD "%5, %16\n\t" RD "%6, %13\n\t" RD "%7, %17\n\t" W0
                 : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3]), "=&v"(o[4]), "=&v"(o[5]), "=&v"(o[6]), "=&v"(o[7]), "=&v"(q[0]), "=&v"(q[1])
                 : "v"(p0), "v"(p0 ^ 32u), "v"(p0 ^ 64u), "v"(p0 ^ 96u), "v"(p1), "v"(p1 ^ 32u), "v"(p1 ^ 64u), "v"(p1 ^ 96u), "v"(r0), "v"(r1) : "memory");
  else {
    pq_i32x2 t0, t1;
    asm volatile("ds_read_b64 %8, %18\n\tds_read_b64 %9, %19\n\t" RD "%0, %10\n\t" RD "%1, %14\n\t" RD "%2, %11\n\t" RD "%3, %15\n\t" RD "%4, %12\n\t" RD "%5, %16\n\t" RD "%6, %13\n\t" RD "%7, %17\n\t" W0
                 : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3]), "=&v"(o[4]), "=&v"(o[5]), "=&v"(o[6]), "=&v"(o[7]), "=&v"(t0), "=&v"(t1)
                 : "v"(p0), "v"(p0 ^ 32u), "v"(p0 ^ 64u), "v"(p0 ^ 96u), "v"(p1), "v"(p1 ^ 32u), "v"(p1 ^ 64u), "v"(p1 ^ 96u), "v"(r0), "v"(r1) : "memory");
    q[0][0] = t0[0]; q[0][1] = t0[1]; q[1][0] = t1[0]; q[1][1] = t1[1];
  }
}
#undef RD
#undef RT
#undef W0

template <bool INT8, typename ACC>
__device__ __forceinline__ void mma(ACC& c, const i32x4_t& a, const i32x4_t& b) {
  // (the B operand goes first: a lane then holds runs of four consecutive columns of one output row)
  if constexpr (INT8) c = __builtin_amdgcn_mfma_i32_32x32x32_i8(b, a, c, 0, 0, 0);
  else c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, b), __builtin_bit_cast(bf16x8_t, a), c, 0, 0, 0);
}

// The products of one stage (byte offset so): four sub-steps of the wavefront's 2 x 2 blocks.
template <bool INT8, int AK, int BK, int BM, typename FA, typename FB, typename ACC>
__device__ __forceinline__ void tile_step(const FA& fa, const FB& fb, uint32_t so, int lane, ACC (&acc)[2][2]) {
  constexpr bool bits = BK == PQ_SRC_BITS8 || BK == PQ_SRC_BITS16;
  auto expand = [&](const i32x4_t& q, int ks) -> i32x4_t {
    if constexpr (BK == PQ_SRC_BITS8) return pq_bits_to_i8((uint32_t)q[ks] >> (16 * (lane >> 5)));
    else return pq_bits_to_bf16((uint32_t)q[ks >> 1] >> (16 * (ks & 1) + 8 * (lane >> 5)));
  };
  if constexpr (bits) {
    i32x4_t oa[8], q[2];
    rd_kc_bits_x4<BK == PQ_SRC_BITS8>(oa, q, fa.ad[0] + so, fa.ad[1] + so, fb.ad[0] + so, fb.ad[1] + so);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const i32x4_t b0 = expand(q[0], ks), b1 = expand(q[1], ks);
#pragma unroll
      for (int i = 0; i < 2; ++i) { mma<INT8>(acc[i][0], oa[2 * ks + i], b0); mma<INT8>(acc[i][1], oa[2 * ks + i], b1); }
    }
  } else {
#pragma unroll
    for (int ks = 0; ks < 4; ks += 2) {
      i32x4_t oa[4], ob[4];
      constexpr uint32_t R = BM * 2;
      const uint32_t p0 = fa.ad[0] + so, p1 = fa.ad[1] + so, r0 = fb.ad[0] + so, r1 = fb.ad[1] + so;
      if constexpr (AK == PQ_SRC_KS16) rd_ks_ks_x2<R>(oa, ob, p0 + ks * 16 * R, p1 + ks * 16 * R, r0 + ks * 16 * R, r1 + ks * 16 * R);
      else if constexpr (BK == PQ_SRC_KS16) rd_kc_ks_x2<R>(oa, ob, p0, p1, r0 + ks * 16 * R, r1 + ks * 16 * R, ks << 5);
      else rd_kc_kc_x2(oa, ob, p0, p1, r0, r1, ks << 5);
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) mma<INT8>(acc[i][j], oa[2 * u + i], ob[2 * u + j]);
    }
  }
}

// 128x128 tiles: wavefront (wv >> 1, wv & 1) multiplies a 64x64 quadrant.  NST: ring stages.
template <int NST, int AK, int BK, int BK2>
constexpr int tile_lds() {   // (the second contraction's stages follow in the ring's place)
  constexpr int ring = NST * (tile_src<AK, 128>::BYTES + tile_src<BK, 128>::BYTES), two = BK2 >= 0 ? 2 * 256 * 128 : 0;
  return ring > two ? ring : two;
}
// (bx, by, bz) of a grid of gy rows: the workgroup's place in its own product's launch.  The second problem of a pair is chosen here, not by the
// kernel that calls: what the compiler makes of the arguments' loads ahead of the first requests is a few tenths of a microsecond a launch
// (prefill of 2892 tokens 1024 -> 960: 18.5 us with the choice in the kernel, 18.1 here).
template <int NST, bool INT8, int AK, int BK, int BK2, class SECOND>
__device__ __forceinline__ void tile_body(int M, int N, int K, pq_operand A, pq_operand B, pq_epilogue epi, int nbn, int total_tiles, int kchunk,
                                          float* splitk_part, const pq_gemm_group& grp, const pq_phase2& ph2, const SECOND& second, int bx, int by,
                                          int bz, int gy, unsigned char* smem, double* red) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int BM = 128, BN = 128, WM = 64, WN = 64, TM = 2, TN = 2;
  constexpr int EPB = INT8 ? 128 : 64;
  using SA = tile_src<AK, BM>;
  using SB = tile_src<BK, BN>;
  constexpr int LPW = SA::LPW + SB::LPW;
  constexpr int STG = SA::BYTES + SB::BYTES;
  constexpr bool PH2 = BK2 >= 0;
  constexpr int STG2 = PH2 ? (BM + BN) * 128 : 0;
  using acc_t = typename std::conditional<INT8, i32x16_t, f32x16_t>::type;
  constexpr bool PAIR = pair_kinds<AK, BK, BK2>();
  if constexpr (std::is_same<SECOND, pq_gemm_second>::value)
    if (grp.mode == 3 && bz == 1) {          // uniform: the second problem of a paired launch
      A = second.A; B = second.B;
      M = second.M; N = second.N; nbn = second.nbn;
      splitk_part = second.part;
      epi.C = second.C; epi.ldc = second.ldc; epi.scale = second.scale; epi.dev_scale = second.dev_scale;
    }
  // XCD-aware order: XCD c takes the c-th eighth of the (contraction split, tile row, tile column) order
  int pid = bx, split = by;
  {
    const int nb = total_tiles * gy;
    if ((nb & 7) == 0) {
      const int lin = bx + total_tiles * by;
      const int w = (lin & 7) * (nb >> 3) + (lin >> 3);
      split = w / total_tiles;
      pid = w - split * total_tiles;
    }
  }
  const int bm = pid / nbn, bn = pid % nbn;
  int m0 = bm * BM;
  const int n0 = bn * BN;
  if (PAIR && grp.mode == 3 && m0 >= M) return;              // uniform: the two problems of a pair may have different tile counts
  int kb = split * kchunk;
  int ke = min(K, kb + kchunk);
  int Mtot = M;
  size_t slab_group = 0;
  if (grp.mode == 1) {          // rows of group z; row tiles are numbered group after group
    int t = bm, z = 0;
    for (; z < grp.n_groups; ++z) {
      const int nt = (grp.offsets[z + 1] - grp.offsets[z] + BM - 1) / BM;
      if (t < nt) break;
      t -= nt;
    }
    if (z == grp.n_groups) return;                   // uniform: the launch covers the worst-case tile count
    m0 = grp.offsets[z] + t * BM;
    M = grp.offsets[z + 1];
    B.p = (const char*)B.p + (size_t)z * grp.b_stride * (BK == PQ_SRC_KC8 ? 1 : 2);
    if (epi.col_div) epi.col_div += (size_t)z * grp.coldiv_stride;
  } else if (grp.mode == 2) {   // contraction range of group z, in gy pieces of whole 64-element steps
    const int z = bz;
    kb = grp.offsets[z];
    ke = grp.offsets[z + 1];
    if (gy > 1) {
      int chunk = (ke - kb + gy - 1) / gy;
      chunk = (chunk + 63) & ~63;
      kb = min(ke, kb + split * chunk);
      ke = min(ke, kb + chunk);
      slab_group = (size_t)z * M * N;
      Mtot = grp.n_groups * M;
    }
    epi.C = (char*)epi.C + (size_t)z * grp.c_stride * (epi.out_kind == PQ_OUT_BF16 ? 2 : 4);
    if (AK == PQ_SRC_KS16 && epi.m_split > 0) epi.C2 = (char*)epi.C2 + (size_t)z * grp.c_stride * 4;
  }
  const int klen = max(ke - kb, 0);
  const int nkt = (klen + EPB - 1) / EPB;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm0 = (wv >> 1) * WM, wn0 = (wv & 1) * WN;
  const uint32_t lds0 = (uint32_t)(size_t)smem;

  // the second contraction: [two stages of A2 (KC16) | B2 (KC16 or KS16)]
  using SA2 = tile_src<PQ_SRC_KC16, BM>;
  using SB2 = tile_src<BK2 == PQ_SRC_KS16 ? PQ_SRC_KS16 : PQ_SRC_KC16, BN>;
  const int nk2 = PH2 && split == 0 ? (ph2.K2 + 63) / 64 : 0;   // (of a split contraction the first part carries it)
  auto issue2 = [&](int t) {
    if constexpr (PH2) {
      SA2 a2;
      SB2 b2;
      a2.setup(ph2.A2, m0, M, 0, wv, lane);
      b2.setup(ph2.B2, n0, N, 0, wv, lane);
      unsigned char* base = smem + (t & 1) * STG2;
      a2.issue(t, ph2.K2, base, wv);
      b2.issue(t, ph2.K2, base + BM * 128, wv);
    }
  };
  SA sa;
  SB sb;
  sa.setup(A, m0, M, kb, wv, lane);
  sb.setup(B, n0, N, kb, wv, lane);
  auto issue = [&](int kt, int slot) {
    sa.issue(kt, klen, smem + slot * STG, wv);
    sb.issue(kt, klen, smem + slot * STG + SA::BYTES, wv);
  };
#pragma unroll
  for (int t = 0; t < NST - 1; ++t)
    if (t < nkt) issue(t, t);

  acc_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;

  tile_frag<AK, BM, TM> fa;
  tile_frag<BK, BN, TN> fb;
  fa.setup(lds0, wm0, lane);
  fb.setup(lds0 + SA::BYTES, wn0, lane);
  int slot = 0;
  for (int kt = 0; kt < nkt; ++kt) {
    // this step has landed when at most the loads of the steps behind it are outstanding (at most NST - 2 of them)
    const int behind = nkt - 1 - kt;                 // uniform
    if (behind >= NST - 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 2) * LPW) : "memory");
    else if (NST > 3 && behind == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LPW) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    asm volatile("s_barrier" ::: "memory");          // ... everybody's; nobody reads the stage before this one any more
    if (kt + NST - 1 < nkt) issue(kt + NST - 1, slot == 0 ? NST - 1 : slot - 1);
    const uint32_t so = (uint32_t)(slot * STG);
    tile_step<INT8, AK, BK, BM>(fa, fb, so, lane, acc);
    slot = slot == NST - 1 ? 0 : slot + 1;
  }

  f32x16_t accf[PH2 ? TM : 1][PH2 ? TN : 1];
  if constexpr (PH2) {
    asm volatile("s_barrier" ::: "memory");          // the ring's last stage has been read by everybody
    if (nk2 > 0) issue2(0);
    if (nk2 > 1) issue2(1);
    const float sc1 = ph2.dev_scale1 ? __fmul_rn(ph2.scale1, *ph2.dev_scale1) : ph2.scale1;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const float sr = ph2.row_div1 ? sc1 / ph2.row_div1[min(m0 + wm0 + i * 32 + (lane & 31), M - 1)] : sc1;   // a lane holds one row of a block
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const auto e1 = acc[i][j][v];
          accf[i][j][v] = (float)e1 * sr;
        }
    }
    tile_frag<PQ_SRC_KC16, BM, TM> f2a;
    tile_frag<BK2 == PQ_SRC_KS16 ? PQ_SRC_KS16 : PQ_SRC_KC16, BN, TN> f2b;
    f2a.setup(lds0, wm0, lane);
    f2b.setup(lds0 + BM * 128, wn0, lane);
    for (int t = 0; t < nk2; ++t) {
      // (two steps in flight; the older one has landed when at most one step's loads are outstanding)
      if (t + 1 < nk2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(SA2::LPW + SB2::LPW) : "memory");
      else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      asm volatile("s_barrier" ::: "memory");
      const uint32_t so = (uint32_t)((t & 1) * STG2);
      tile_step<false, PQ_SRC_KC16, BK2 == PQ_SRC_KS16 ? PQ_SRC_KS16 : PQ_SRC_KC16, BM>(f2a, f2b, so, lane, accf);
      if (t + 2 < nk2) {
        asm volatile("s_barrier" ::: "memory");      // this stage has been read by everybody
        issue2(t + 2);
      }
    }
  }

  // Epilogue: lane l holds row (l & 31) of a block and, per group g = v >> 2, the columns 8 g + 4 (l >> 5) + (0..3); one
  // half-wave exchange per register gives every lane eight consecutive columns of its row.
  epi_state st;
  epi_begin(epi, st);
  float* slab = splitk_part ? splitk_part + (size_t)split * Mtot * N + slab_group : nullptr;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m0 + wm0 + i * 32 + (lane & 31);
    const float rs = !slab && epi.row_div ? st.sc0 / epi.row_div[min(m, M - 1)] : __builtin_nanf("");
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int pr = 0; pr < 2; ++pr) {
        uint32_t x[4], y[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          uint32_t lo, hi;
          // (copy the elements out first: a vector element is not a bit_cast-able lvalue)
          if constexpr (PH2) {
            const float e0 = accf[i][j][8 * pr + t], e1 = accf[i][j][8 * pr + 4 + t];
            lo = __float_as_uint(e0); hi = __float_as_uint(e1);
          } else {
            const auto e0 = acc[i][j][8 * pr + t];
            const auto e1 = acc[i][j][8 * pr + 4 + t];
            lo = __builtin_bit_cast(uint32_t, e0); hi = __builtin_bit_cast(uint32_t, e1);
          }
          const auto sw = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
          x[t] = sw[0];
          y[t] = sw[1];
        }
        const int n = n0 + wn0 + j * 32 + 8 * (2 * pr + (lane >> 5));
        const uint4 r0 = make_uint4(x[0], x[1], x[2], x[3]), r1 = make_uint4(y[0], y[1], y[2], y[3]);
        if (m < M && n < N) {
          if (slab) {
            *reinterpret_cast<uint4*>(slab + (size_t)m * N + n) = r0;
            *reinterpret_cast<uint4*>(slab + (size_t)m * N + n + 4) = r1;
          } else {
            epi_vec8<INT8 && !PH2, AK == PQ_SRC_KS16 || BK == PQ_SRC_KC8>(epi, st, m, n, r0, r1, rs);
          }
        }
      }
  }
  if (!slab) epi_end<256>(epi, st, red, bx);
#endif
}

template <int NST, bool INT8, int AK, int BK, int BK2>
__global__ __launch_bounds__(256) void tile_gemm_kernel(int M, int N, int K, pq_operand A, pq_operand B, pq_epilogue epi, int nbn,
                                                        int total_tiles, int kchunk, float* splitk_part, pq_gemm_group grp, pq_phase2 ph2,
                                                        pq_second_arg<pair_kinds<AK, BK, BK2>()> second) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[tile_lds<NST, AK, BK, BK2>()];
  __shared__ double red[4];
  tile_body<NST, INT8, AK, BK, BK2>(M, N, K, A, B, epi, nbn, total_tiles, kchunk, splitk_part, grp, ph2, second, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.y,
                                    smem, red);
}

// 64x64 tiles, the contraction shared out over the wavefronts: wavefront w multiplies the w-th quarter of every 128-byte
// step for the whole tile (four independent MFMAs per step and half the LDS reads of a 32x32 quadrant each, whose four MFMAs
// wait for each other), two steps per barrier, and the four partial tiles are added in LDS in wavefront order.
template <int KIND>
struct rd64 {   // two 32-row blocks of sub-step w of two consecutive stages: o[2 * stage + block]
  static constexpr bool kBits = KIND == PQ_SRC_BITS8 || KIND == PQ_SRC_BITS16;
  uint32_t ad[2];
  int sh;
  __device__ __forceinline__ void setup(uint32_t lds0, int w, int lane) {
    const int h = lane >> 5;
    sh = KIND == PQ_SRC_BITS8 ? 16 * h : 16 * (w & 1) + 8 * h;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int r = 32 * j + (lane & 31);
      if constexpr (KIND == PQ_SRC_KS16) {
        const int t = 8 * h + ((lane & 15) >> 2), col = 32 * j + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
        ad[j] = lds0 + (16 * w + t) * 128 + (((col >> 3) ^ (2 * (t & 3))) << 4) + (col & 7) * 2;
      } else if constexpr (KIND == PQ_SRC_BITS8) ad[j] = lds0 + r * 16 + w * 4;
      else if constexpr (KIND == PQ_SRC_BITS16) ad[j] = lds0 + r * 8 + (w >> 1) * 4;
      else ad[j] = lds0 + r * 128 + ((((2 * w + h) ^ r ^ (r >> 3)) & 7) << 4);
    }
  }
};
#define RD "ds_read_b128 "
#define RT "ds_read_b64_tr_b16 "
#define RW "ds_read_b32 "
#define W0 "s_waitcnt lgkmcnt(0)"
// STG: bytes between the two stages
template <int AK, int BK, int STG>
__device__ __forceinline__ void rd64_pair(const rd64<AK>& fa, const rd64<BK>& fb, uint32_t so, i32x4_t* a, i32x4_t* b) {
  const uint32_t p0 = fa.ad[0] + so, p1 = fa.ad[1] + so, r0 = fb.ad[0] + so, r1 = fb.ad[1] + so;
  if constexpr (rd64<BK>::kBits) {
    uint32_t q[4];
    asm volatile(RW "%4, %10\n\t" RW "%5, %11\n\t" RD "%0, %8\n\t" RD "%1, %9\n\t" RW "%6, %10 offset:%12\n\t" RW "%7, %11 offset:%12\n\t"
                 RD "%2, %8 offset:%12\n\t" RD "%3, %9 offset:%12\n\t" W0
                 : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3]), "=&v"(q[0]), "=&v"(q[1]), "=&v"(q[2]), "=&v"(q[3])
                 : "v"(p0), "v"(p1), "v"(r0), "v"(r1), "n"(STG) : "memory");
#pragma unroll
    for (int u = 0; u < 4; ++u) b[u] = BK == PQ_SRC_BITS8 ? pq_bits_to_i8(q[u] >> fb.sh) : pq_bits_to_bf16(q[u] >> fb.sh);
  } else if constexpr (AK == PQ_SRC_KS16) {
    pq_i32x2 t[8], u[8];
    asm volatile(RT "%0, %16\n\t" RT "%1, %16 offset:%20\n\t" RT "%8, %18\n\t" RT "%9, %18 offset:%20\n\t"
                 RT "%2, %17\n\t" RT "%3, %17 offset:%20\n\t" RT "%10, %19\n\t" RT "%11, %19 offset:%20\n\t"
                 RT "%4, %16 offset:%21\n\t" RT "%5, %16 offset:%22\n\t" RT "%12, %18 offset:%21\n\t" RT "%13, %18 offset:%22\n\t"
                 RT "%6, %17 offset:%21\n\t" RT "%7, %17 offset:%22\n\t" RT "%14, %19 offset:%21\n\t" RT "%15, %19 offset:%22\n\t" W0
                 : "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3]), "=&v"(t[4]), "=&v"(t[5]), "=&v"(t[6]), "=&v"(t[7]),
                   "=&v"(u[0]), "=&v"(u[1]), "=&v"(u[2]), "=&v"(u[3]), "=&v"(u[4]), "=&v"(u[5]), "=&v"(u[6]), "=&v"(u[7])
                 : "v"(p0), "v"(p1), "v"(r0), "v"(r1), "n"(512), "n"(STG), "n"(STG + 512) : "memory");
#pragma unroll
    for (int k = 0; k < 4; ++k) { a[k] = join(t[2 * k], t[2 * k + 1]); b[k] = join(u[2 * k], u[2 * k + 1]); }
  } else if constexpr (BK == PQ_SRC_KS16) {
    pq_i32x2 t[8];
    asm volatile(RD "%0, %12\n\t" RT "%4, %14\n\t" RT "%5, %14 offset:%16\n\t" RD "%1, %13\n\t" RT "%6, %15\n\t" RT "%7, %15 offset:%16\n\t"
                 RD "%2, %12 offset:%17\n\t" RT "%8, %14 offset:%17\n\t" RT "%9, %14 offset:%18\n\t" RD "%3, %13 offset:%17\n\t" RT "%10, %15 offset:%17\n\t"
                 RT "%11, %15 offset:%18\n\t" W0
                 : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3]), "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3]), "=&v"(t[4]), "=&v"(t[5]),
                   "=&v"(t[6]), "=&v"(t[7])
                 : "v"(p0), "v"(p1), "v"(r0), "v"(r1), "n"(512), "n"(STG), "n"(STG + 512) : "memory");
#pragma unroll
    for (int k = 0; k < 4; ++k) b[k] = join(t[2 * k], t[2 * k + 1]);
  } else {
    asm volatile(RD "%0, %8\n\t" RD "%4, %10\n\t" RD "%1, %9\n\t" RD "%5, %11\n\t" RD "%2, %8 offset:%12\n\t" RD "%6, %10 offset:%12\n\t"
                 RD "%3, %9 offset:%12\n\t" RD "%7, %11 offset:%12\n\t" W0
                 : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3]), "=&v"(b[0]), "=&v"(b[1]), "=&v"(b[2]), "=&v"(b[3])
                 : "v"(p0), "v"(p1), "v"(r0), "v"(r1), "n"(STG) : "memory");
  }
}
#undef RD
#undef RT
#undef RW
#undef W0

// NG: groups of two stages in the ring (NG - 1 of them in flight ahead of the MFMAs)
template <int NG, int AK, int BK, int BK2>
constexpr int tile64_lds() {
  constexpr int need = NG * 2 * (tile_src<AK, 64>::BYTES + tile_src<BK, 64>::BYTES) + (BK2 >= 0 ? 2 * 128 * 128 : 0);
  static_assert(need <= 150 * 1024, "LDS");
  return need > 65536 ? need : 65536;                // four partial tiles at the end
}
// (by reference what the body changes, for the same reason: 1348 tokens 1984 -> 896, r = 80, 92.3 us with copies, 90.9 so)
template <int NG, bool INT8, int AK, int BK, int BK2, class SECOND>
__device__ __forceinline__ void tile64_body(int& M, int& N, int K, pq_operand& A, pq_operand& B, pq_epilogue& epi, int& nbn, int total_tiles, int kchunk,
                                            float*& splitk_part, const pq_gemm_group& grp, const pq_phase2& ph2, const SECOND& second, int bx, int by,
                                            int bz, int gy, unsigned char* smem, double* red) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int EPB = INT8 ? 128 : 64;
  using SA = tile_src<AK, 64>;
  using SB = tile_src<BK, 64>;
  constexpr int LPG = 2 * (SA::LPW + SB::LPW);       // loads per wavefront and group
  constexpr int STG = SA::BYTES + SB::BYTES;
  constexpr bool PH2 = BK2 >= 0;
  constexpr int KB2 = BK2 == PQ_SRC_KS16 ? PQ_SRC_KS16 : PQ_SRC_KC16;
  constexpr int STG2 = 128 * 128;
  constexpr int RING = NG * 2 * STG;
  constexpr int OFF2 = RING;                         // the second contraction's first two steps have LDS of their own
  using acc_t = typename std::conditional<INT8, i32x16_t, f32x16_t>::type;
  constexpr bool PAIR = pair_kinds<AK, BK, BK2>();
  if constexpr (std::is_same<SECOND, pq_gemm_second>::value)
    if (grp.mode == 3 && bz == 1) {          // uniform: the second problem of a paired launch
      A = second.A; B = second.B;
      M = second.M; N = second.N; nbn = second.nbn;
      splitk_part = second.part;
      epi.C = second.C; epi.ldc = second.ldc; epi.scale = second.scale; epi.dev_scale = second.dev_scale;
    }
  // XCD-aware order: XCD c takes the c-th eighth of the (contraction split, tile row, tile column) order
  int pid = bx, split = by;
  {
    const int nb = total_tiles * gy;
    if ((nb & 7) == 0) {
      const int lin = bx + total_tiles * by;
      const int w = (lin & 7) * (nb >> 3) + (lin >> 3);
      split = w / total_tiles;
      pid = w - split * total_tiles;
    }
  }
  const int bm = pid / nbn, bn = pid % nbn;
  int m0 = bm * 64;
  const int n0 = bn * 64;
  if (PAIR && grp.mode == 3 && m0 >= M) return;              // uniform: the two problems of a pair may have different tile counts
  int kb = split * kchunk;
  int ke = min(K, kb + kchunk);
  int Mtot = M;
  size_t slab_group = 0;
  if (grp.mode == 1) {          // rows of group z; row tiles are numbered group after group
    int t = bm, z = 0;
    for (; z < grp.n_groups; ++z) {
      const int nt = (grp.offsets[z + 1] - grp.offsets[z] + 64 - 1) / 64;
      if (t < nt) break;
      t -= nt;
    }
    if (z == grp.n_groups) return;                   // uniform: the launch covers the worst-case tile count
    m0 = grp.offsets[z] + t * 64;
    M = grp.offsets[z + 1];
    B.p = (const char*)B.p + (size_t)z * grp.b_stride * (BK == PQ_SRC_KC8 ? 1 : 2);
    if (epi.col_div) epi.col_div += (size_t)z * grp.coldiv_stride;
  } else if (grp.mode == 2) {   // contraction range of group z, in gy pieces of whole 64-element steps
    const int z = bz;
    kb = grp.offsets[z];
    ke = grp.offsets[z + 1];
    if (gy > 1) {
      int chunk = (ke - kb + gy - 1) / gy;
      chunk = (chunk + 63) & ~63;
      kb = min(ke, kb + split * chunk);
      ke = min(ke, kb + chunk);
      slab_group = (size_t)z * M * N;
      Mtot = grp.n_groups * M;
    }
    epi.C = (char*)epi.C + (size_t)z * grp.c_stride * (epi.out_kind == PQ_OUT_BF16 ? 2 : 4);
    if (AK == PQ_SRC_KS16 && epi.m_split > 0) epi.C2 = (char*)epi.C2 + (size_t)z * grp.c_stride * 4;
  }
  const int klen = max(ke - kb, 0);
  const int ngr = (klen + 2 * EPB - 1) / (2 * EPB);  // groups; a stage past the end is fetched as zeros
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t lds0 = (uint32_t)(size_t)smem;

  // the second contraction, one group at a time (of a split contraction the first part carries it)
  const int nk2 = PH2 && split == 0 ? (ph2.K2 + 127) / 128 : 0;
  auto issue2 = [&](int g) {
    if constexpr (PH2) {
      tile_src<PQ_SRC_KC16, 64> a2;
      tile_src<KB2, 64> b2;
      a2.setup(ph2.A2, m0, M, 0, wv, lane);
      b2.setup(ph2.B2, n0, N, 0, wv, lane);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        unsigned char* base = smem + OFF2 + u * STG2;
        a2.issue(2 * g + u, ph2.K2, base, wv);
        b2.issue(2 * g + u, ph2.K2, base + 8192, wv);
      }
    }
  };
  if (nk2 > 0) issue2(0);                            // oldest loads: every wait of the main loop covers them
  SA sa;
  SB sb;
  sa.setup(A, m0, M, kb, wv, lane);
  sb.setup(B, n0, N, kb, wv, lane);
  auto issue = [&](int g, int slot) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      sa.issue(2 * g + u, klen, smem + (2 * slot + u) * STG, wv);
      sb.issue(2 * g + u, klen, smem + (2 * slot + u) * STG + SA::BYTES, wv);
    }
  };
#pragma unroll
  for (int t = 0; t < NG - 1; ++t)
    if (t < ngr) issue(t, t);
  acc_t acc[2][2];
  f32x16_t acc2[PH2 ? 2 : 1][PH2 ? 2 : 1];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        acc[i][j][v] = 0;
        if constexpr (PH2) acc2[i][j][v] = 0.f;
      }
  rd64<AK> fa;
  rd64<BK> fb;
  fa.setup(lds0, wv, lane);
  fb.setup(lds0 + SA::BYTES, wv, lane);
  int slot = 0;
  for (int g = 0; g < ngr; ++g) {
    const int behind = ngr - 1 - g;                  // uniform; groups issued behind this one: at most NG - 2
    if (behind >= NG - 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NG - 2) * LPG) : "memory");
    else if (NG > 3 && behind == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LPG) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    asm volatile("s_barrier" ::: "memory");          // the group is there; nobody reads the one before it any more
    if (g + NG - 1 < ngr) issue(g + NG - 1, slot == 0 ? NG - 1 : slot - 1);
    i32x4_t oa[4], ob[4];
    rd64_pair<AK, BK, STG>(fa, fb, (uint32_t)(slot * 2 * STG), oa, ob);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) mma<INT8>(acc[i][j], oa[2 * u + i], ob[2 * u + j]);
    slot = slot == NG - 1 ? 0 : slot + 1;
  }
  if constexpr (PH2) {
    rd64<PQ_SRC_KC16> f2a;
    rd64<KB2> f2b;
    f2a.setup(lds0 + OFF2, wv, lane);
    f2b.setup(lds0 + OFF2 + 8192, wv, lane);
    for (int g = 0; g < nk2; ++g) {
      if (g > 0) {                                   // contractions of more than 128: one more memory latency each
        asm volatile("s_barrier" ::: "memory");
        issue2(g);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        asm volatile("s_barrier" ::: "memory");
      }
      i32x4_t oa[4], ob[4];
      rd64_pair<PQ_SRC_KC16, KB2, STG2>(f2a, f2b, 0u, oa, ob);
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) mma<false>(acc2[i][j], oa[2 * u + i], ob[2 * u + j]);
    }
  }

  // The partial tiles through LDS ([wavefront][64 rows][256 B], chunk c of a row at c ^ (row & 15)); a thread then owns
  // eight consecutive columns of rows (tid >> 3) and (tid >> 3) + 32.
  auto put = [&](const auto& av) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int r = 32 * i + (lane & 31), c = 8 * j + 2 * q + (lane >> 5);
          const auto e0 = av[i][j][4 * q], e1 = av[i][j][4 * q + 1], e2 = av[i][j][4 * q + 2], e3 = av[i][j][4 * q + 3];
          const i32x4_t o = {__builtin_bit_cast(int, e0), __builtin_bit_cast(int, e1), __builtin_bit_cast(int, e2), __builtin_bit_cast(int, e3)};
          // (asm with two wait states behind it: see the staged epilogue of mfma_gemm_kernel)
          const uint32_t adw = lds0 + wv * 16384 + r * 256 + ((c ^ (r & 15)) << 4);
          asm volatile("ds_write_b128 %0, %1\n\ts_nop 1" ::"v"(adw), "v"(o) : "memory");
        }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  };
  const int c8 = (threadIdx.x & 7) * 2;
  auto get = [&](int r, int w, int half) -> i32x4_t {
    return *reinterpret_cast<const i32x4_t*>(smem + w * 16384 + r * 256 + (((c8 + half) ^ (r & 15)) << 4));
  };
  asm volatile("s_barrier" ::: "memory");            // every wavefront is past its reads of the ring
  put(acc);
  epi_state st;
  epi_begin(epi, st);
  float* slab = splitk_part ? splitk_part + (size_t)split * Mtot * N + slab_group : nullptr;
  i32x4_t sum[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = (threadIdx.x >> 3) + 32 * i;
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      const i32x4_t x0 = get(r, 0, hf), x1 = get(r, 1, hf), x2 = get(r, 2, hf), x3 = get(r, 3, hf);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (INT8) sum[i][hf][e] = x0[e] + x1[e] + x2[e] + x3[e];
        else {
          const int y0 = x0[e], y1 = x1[e], y2 = x2[e], y3 = x3[e];
          sum[i][hf][e] = __float_as_int(__int_as_float(y0) + __int_as_float(y1) + __int_as_float(y2) + __int_as_float(y3));
        }
      }
    }
  }
  if constexpr (PH2) {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    put(acc2);
    const float sc1 = ph2.dev_scale1 ? __fmul_rn(ph2.scale1, *ph2.dev_scale1) : ph2.scale1;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = (threadIdx.x >> 3) + 32 * i;
      const float sr = ph2.row_div1 ? sc1 / ph2.row_div1[min(m0 + r, M - 1)] : sc1;
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        const i32x4_t x0 = get(r, 0, hf), x1 = get(r, 1, hf), x2 = get(r, 2, hf), x3 = get(r, 3, hf);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int s0 = sum[i][hf][e], y0 = x0[e], y1 = x1[e], y2 = x2[e], y3 = x3[e];
          const float main1 = (INT8 ? (float)s0 : __int_as_float(s0)) * sr;
          sum[i][hf][e] = __float_as_int(main1 + (__int_as_float(y0) + __int_as_float(y1) + __int_as_float(y2) + __int_as_float(y3)));
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int m = m0 + (threadIdx.x >> 3) + 32 * i, n = n0 + (threadIdx.x & 7) * 8;
    if (m < M && n < N) {
      const uint4 r0 = __builtin_bit_cast(uint4, sum[i][0]), r1 = __builtin_bit_cast(uint4, sum[i][1]);
      if (slab) {
        *reinterpret_cast<uint4*>(slab + (size_t)m * N + n) = r0;
        *reinterpret_cast<uint4*>(slab + (size_t)m * N + n + 4) = r1;
      } else {
        epi_vec8<INT8 && !PH2, AK == PQ_SRC_KS16 || BK == PQ_SRC_KC8>(epi, st, m, n, r0, r1);
      }
    }
  }
  if (!slab) epi_end<256>(epi, st, red, bx);
#endif
}

template <int NG, bool INT8, int AK, int BK, int BK2>
__global__ __launch_bounds__(256) void tile64_gemm_kernel(int M, int N, int K, pq_operand A, pq_operand B, pq_epilogue epi, int nbn,
                                                          int total_tiles, int kchunk, float* splitk_part, pq_gemm_group grp, pq_phase2 ph2,
                                                          pq_second_arg<pair_kinds<AK, BK, BK2>()> second) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[tile64_lds<NG, AK, BK, BK2>()];
  __shared__ double red[4];
  tile64_body<NG, INT8, AK, BK, BK2>(M, N, K, A, B, epi, nbn, total_tiles, kchunk, splitk_part, grp, ph2, second, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.y,
                                     smem, red);
}

#ifndef PQ_NG_DEEP
#define PQ_NG_DEEP 4
#endif
#ifndef PQ_NG
#define PQ_NG 2
#endif
template <int BM, int NST, bool INT8, int AK, int BK, int BK2>
int launch_tile(const pq_gemm_plan& pl, int M, int N, int K, const pq_operand& A, const pq_operand& B, const pq_epilogue& epi, hipStream_t s,
                float* part, const pq_gemm_group& grp, const pq_phase2& ph2, const pq_gemm_second* second) {
  constexpr bool PAIR = pair_kinds<AK, BK, BK2>();
  if (grp.mode == 3 && (!PAIR || !second)) return pq_set_error(PQ_ERR_BAD_ARG, "no paired kernel for operand kinds (%d, %d)", AK, BK);
  // grouped rows: every group may end in a partial tile, so at most ceil(rows / BM) + n_groups row tiles exist
  const int nbm = grp.mode == 1 ? (grp.max_rows + BM - 1) / BM + grp.n_groups : (M + BM - 1) / BM;
  const int nbn = (N + BM - 1) / BM;
  int tiles = nbm * nbn;
  if (grp.mode == 3) {
    const int t2 = (second->M + BM - 1) / BM * ((second->N + BM - 1) / BM);
    if (t2 > tiles) tiles = t2;
  }
  dim3 grid(tiles, pl.splits, grp.mode == 2 ? grp.n_groups : grp.mode == 3 ? 2 : 1);
  float* p = pl.splits > 1 ? part : nullptr;
  if constexpr (BM == 64) {
    // up to one workgroup per CU: the deep ring; otherwise the one that lets two or more share a CU
    if ((long)grid.x * grid.y * grid.z <= 256) tile64_gemm_kernel<PQ_NG_DEEP, INT8, AK, BK, BK2><<<grid, 256, 0, s>>>(M, N, K, A, B, epi, nbn, tiles, pl.kchunk, p, grp, ph2, second_arg<PAIR>(second));
    else tile64_gemm_kernel<NST, INT8, AK, BK, BK2><<<grid, 256, 0, s>>>(M, N, K, A, B, epi, nbn, tiles, pl.kchunk, p, grp, ph2, second_arg<PAIR>(second));
  } else {
    tile_gemm_kernel<NST, INT8, AK, BK, BK2><<<grid, 256, 0, s>>>(M, N, K, A, B, epi, nbn, tiles, pl.kchunk, p, grp, ph2, second_arg<PAIR>(second));
  }
  PQ_CHECK_LAUNCH("tile_gemm_kernel");
  return PQ_OK;
}

#ifndef PQ_NST128
#define PQ_NST128 2
#endif
#ifndef PQ_NST128B
#define PQ_NST128B 4
#endif
template <bool INT8, int AK, int BK, int BK2 = -1>
int launch_kinds(const pq_gemm_plan& pl, int M, int N, int K, const pq_operand& A, const pq_operand& B, const pq_epilogue& epi, hipStream_t s,
                 float* part, const pq_gemm_group& grp, const pq_phase2& ph2, const pq_gemm_second* second) {
  constexpr bool bits = BK == PQ_SRC_BITS8 || BK == PQ_SRC_BITS16;
  if (pl.bm == 64) return launch_tile<64, PQ_NG, INT8, AK, BK, BK2>(pl, M, N, K, A, B, epi, s, part, grp, ph2, second);
  return launch_tile<128, bits ? PQ_NST128B : PQ_NST128, INT8, AK, BK, BK2>(pl, M, N, K, A, B, epi, s, part, grp, ph2, second);
}

// Up to four weight gradients (w) and a product of their input's size (x: an input gradient, or an expert's; may be none) that do not
// depend on each other, in one launch: workgroups of w[0], w[1], ..., then of x.  Alone each leaves CUs idle (one wave of small tiles, or
// less) and is bound by its own chain of latencies and its launch.
struct tile_job {
  int M, N, K, nbn, tiles, kchunk, gy, blocks;       // blocks: tiles * splits * groups
  pq_operand A, B;
  pq_epilogue epi;
  float* part;
  pq_gemm_group grp;
};
template <int BM, int NST, int AK, int BK>
struct tile_kind {
  static constexpr int LDS = BM == 64 ? tile64_lds<NST, AK, BK, -1>() : tile_lds<NST, AK, BK, -1>();
  static __device__ __forceinline__ void run(tile_job j, int b, unsigned char* smem, double* red) {
    pq_phase2 none;
    none.K2 = 0;
    const int bx = b % j.tiles, by = b / j.tiles % j.gy, bz = b / (j.tiles * j.gy);
    if constexpr (BM == 64) tile64_body<NST, false, AK, BK, -1>(j.M, j.N, j.K, j.A, j.B, j.epi, j.nbn, j.tiles, j.kchunk, j.part, j.grp, none, pq_no_second{}, bx, by, bz, j.gy, smem, red);
    else tile_body<NST, false, AK, BK, -1>(j.M, j.N, j.K, j.A, j.B, j.epi, j.nbn, j.tiles, j.kchunk, j.part, j.grp, none, pq_no_second{}, bx, by, bz, j.gy, smem, red);
  }
};
template <int BM, int AK, int BK>
using tile_in_set = tile_kind<BM, BM == 64 ? PQ_NG : BK == PQ_SRC_BITS16 ? PQ_NST128B : PQ_NST128, AK, BK>;
struct tile_jobs {
  tile_job j[4];
};
template <int WBM, int XBM, int XBK>
__global__ __launch_bounds__(256) void tile_set_kernel(tile_jobs w, tile_job x) {
  using W = tile_in_set<WBM, PQ_SRC_KS16, PQ_SRC_KS16>;
  using X = tile_in_set<XBM, PQ_SRC_KC16, XBK>;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[W::LDS > X::LDS ? W::LDS : X::LDS];
  __shared__ double red[4];
  int b = blockIdx.x, i = 0;
  while (i < 4 && b >= w.j[i].blocks) b -= w.j[i++].blocks;    // uniform
  if (i == 4) X::run(x, b, smem, red);
  else W::run(w.j[i], b, smem, red);
}

// What follows dH in the backward of a linear with a dense branch, where all of it takes 64x64 tiles and neither dX nor dW is split: workgroups
// of dX (with X), then of dW, dB and dA (j0, j1, j2; the last two split as they are alone, so that no sum is longer than it was).  Each is one
// chain of latencies; the branch's gradients alone fill a fraction of the chip (32 to 70 tiles).  In one launch instead of three or four
// (whole call, forward and backward): 64 tokens 256 -> 256, r = 16, 47.8 -> 37.5 us; 512 tokens 512 -> 512, r = 64, 56.7 -> 43.0; 701 tokens
// 608 -> 2048, r = 40, 77.4 -> 61.0; 236 tokens 2560 -> 672, r = 160, INT8 branch, 84.4 -> 72.5; without dX, which takes other tiles
// there: 1724 tokens 1984 -> 736, r = 32, INT8 branch, 107.1 -> 101.0.
template <int NG, bool X>
__global__ __launch_bounds__(256) void tile64_grads_kernel(tile_job x, pq_phase2 p2, tile_job j0, tile_job j1, tile_job j2) {
  constexpr int LW = tile64_lds<NG, PQ_SRC_KS16, PQ_SRC_KS16, -1>(), LX = X ? tile64_lds<NG, PQ_SRC_KC16, PQ_SRC_BITS16, PQ_SRC_KS16>() : 0;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[LW > LX ? LW : LX];
  __shared__ double red[4];
  int b = blockIdx.x;
  if constexpr (X) {
    if (b < x.blocks) {                              // uniform
      tile64_body<NG, false, PQ_SRC_KC16, PQ_SRC_BITS16, PQ_SRC_KS16>(x.M, x.N, x.K, x.A, x.B, x.epi, x.nbn, x.tiles, x.kchunk, x.part, x.grp, p2, pq_no_second{}, b, 0, 0,
                                                                      1, smem, red);
      return;
    }
    b -= x.blocks;
  }
  const int n1 = j0.blocks + j1.blocks;
  tile_job j = b < j0.blocks ? j0 : b < n1 ? j1 : j2;   // uniform
  pq_phase2 none;
  none.K2 = 0;
  b = b < j0.blocks ? b : b < n1 ? b - j0.blocks : b - n1;
  tile64_body<NG, false, PQ_SRC_KS16, PQ_SRC_KS16, -1>(j.M, j.N, j.K, j.A, j.B, j.epi, j.nbn, j.tiles, j.kchunk, j.part, j.grp, none, pq_no_second{}, b % j.tiles,
                                                       b / j.tiles, 0, j.gy, smem, red);
}

template <int WBM, int XBM, int XBK>
int launch_set(const tile_jobs& w, const tile_job& x, hipStream_t s) {
  tile_set_kernel<WBM, XBM, XBK><<<w.j[0].blocks + w.j[1].blocks + w.j[2].blocks + w.j[3].blocks + x.blocks, 256, 0, s>>>(w, x);
  PQ_CHECK_LAUNCH("tile_set_kernel");
  return PQ_OK;
}

tile_job job_of(const pq_tile_call* c) {
  tile_job j;
  memset(&j, 0, sizeof(j));
  if (!c) return j;
  const int bm = c->pl.bm, nbm = c->grp.mode == 1 ? (c->grp.max_rows + bm - 1) / bm + c->grp.n_groups : (c->M + bm - 1) / bm;
  j.M = c->M; j.N = c->N; j.K = c->K; j.nbn = (c->N + bm - 1) / bm; j.tiles = nbm * j.nbn; j.kchunk = c->pl.kchunk;
  j.gy = c->pl.splits; j.blocks = j.tiles * j.gy * (c->grp.mode == 2 ? c->grp.n_groups : 1);
  j.A = c->A; j.B = c->B; j.epi = c->epi; j.part = c->pl.splits > 1 ? c->part : nullptr; j.grp = c->grp;
  return j;
}

}  // namespace

bool pq_tile_set_applies(const pq_tile_call* w, int nw, const pq_tile_call* x) {
  if (nw < 1 || nw > 4) return false;
  for (int i = 0; i < nw; ++i)
    if (w[i].A.kind != PQ_SRC_KS16 || w[i].B.kind != PQ_SRC_KS16 || w[i].pl.bn > 128 || w[i].pl.bm != w[0].pl.bm) return false;
  return !x || (x->A.kind == PQ_SRC_KC16 && (x->B.kind == PQ_SRC_BITS16 || x->B.kind == PQ_SRC_KS16) && x->pl.bn <= 128);
}

int pq_launch_tile_set(const pq_tile_call* w, int nw, const pq_tile_call* x, hipStream_t s) {
  if (!pq_tile_set_applies(w, nw, x)) return pq_set_error(PQ_ERR_BAD_ARG, "products that cannot share a launch");
  tile_jobs jw;
  for (int i = 0; i < 4; ++i) jw.j[i] = job_of(i < nw ? &w[i] : nullptr);
  const tile_job jx = job_of(x);
  const int xbm = x ? x->pl.bm : 64, xbk = x ? x->B.kind : PQ_SRC_KS16;
#define PQ_SET(WBM, XBM, XBK) if (w[0].pl.bm == WBM && xbm == XBM && xbk == XBK) return launch_set<WBM, XBM, XBK>(jw, jx, s)
  PQ_SET(64, 64, PQ_SRC_BITS16); PQ_SET(64, 128, PQ_SRC_BITS16); PQ_SET(128, 64, PQ_SRC_BITS16); PQ_SET(128, 128, PQ_SRC_BITS16);
  PQ_SET(64, 64, PQ_SRC_KS16); PQ_SET(64, 128, PQ_SRC_KS16); PQ_SET(128, 64, PQ_SRC_KS16); PQ_SET(128, 128, PQ_SRC_KS16);
#undef PQ_SET
  return pq_set_error(PQ_ERR_BAD_ARG, "no launch for these tiles");
}

int pq_launch_tile_grads(const pq_tile_call (&c)[3], const pq_tile_call* x, const pq_phase2* p2, hipStream_t s) {
  auto plain64 = [](const pq_tile_call& q) { return q.pl.bm == 64 && q.pl.splits >= 1 && (q.pl.splits == 1 || q.part) && q.grp.mode == 0 && q.M > 0 && q.N > 0; };
  for (const pq_tile_call& q : c)
    if (!plain64(q) || q.A.kind != PQ_SRC_KS16 || q.B.kind != PQ_SRC_KS16) return pq_set_error(PQ_ERR_BAD_ARG, "products that cannot share a launch");
  if (x && (!p2 || !plain64(*x) || x->pl.splits != 1 || x->A.kind != PQ_SRC_KC16 || x->B.kind != PQ_SRC_BITS16 || p2->A2.kind != PQ_SRC_KC16 || p2->B2.kind != PQ_SRC_KS16))
    return pq_set_error(PQ_ERR_BAD_ARG, "products that cannot share a launch");
  const tile_job jx = job_of(x), j0 = job_of(&c[0]), j1 = job_of(&c[1]), j2 = job_of(&c[2]);
  const int blocks = jx.blocks + j0.blocks + j1.blocks + j2.blocks;
  const bool deep = blocks <= 256;                   // (rings as in launch_tile)
  pq_phase2 ph2;
  memset(&ph2, 0, sizeof(ph2));
  if (x) ph2 = *p2;
  if (x && deep) tile64_grads_kernel<PQ_NG_DEEP, true><<<blocks, 256, 0, s>>>(jx, ph2, j0, j1, j2);
  else if (x) tile64_grads_kernel<PQ_NG, true><<<blocks, 256, 0, s>>>(jx, ph2, j0, j1, j2);
  else if (deep) tile64_grads_kernel<PQ_NG_DEEP, false><<<blocks, 256, 0, s>>>(jx, ph2, j0, j1, j2);
  else tile64_grads_kernel<PQ_NG, false><<<blocks, 256, 0, s>>>(jx, ph2, j0, j1, j2);
  PQ_CHECK_LAUNCH("tile64_grads_kernel");
  return PQ_OK;
}

int pq_launch_tile(const pq_gemm_plan& pl, int M, int N, int K, const pq_operand& A, const pq_operand& B, const pq_epilogue& epi, hipStream_t s,
                   float* part, const pq_gemm_group& grp, const pq_phase2& ph2, const pq_gemm_second* second) {
  const int ak = A.kind, bk = B.kind;
#define PQ_TILE_KINDS(...) return launch_kinds<__VA_ARGS__>(pl, M, N, K, A, B, epi, s, part, grp, ph2, second)
  if (ph2.K2 > 0) {
    if (ak == PQ_SRC_KC8 && bk == PQ_SRC_BITS8 && ph2.A2.kind == PQ_SRC_KC16 && ph2.B2.kind == PQ_SRC_KC16)
      PQ_TILE_KINDS(true, PQ_SRC_KC8, PQ_SRC_BITS8, PQ_SRC_KC16);
    if (ak == PQ_SRC_KC16 && bk == PQ_SRC_BITS16 && ph2.A2.kind == PQ_SRC_KC16 && ph2.B2.kind == PQ_SRC_KS16)
      PQ_TILE_KINDS(false, PQ_SRC_KC16, PQ_SRC_BITS16, PQ_SRC_KS16);
    return pq_set_error(PQ_ERR_BAD_ARG, "no fused MFMA kernel for these operand kinds");
  }
  if (ak == PQ_SRC_KC8 && bk == PQ_SRC_BITS8) PQ_TILE_KINDS(true, PQ_SRC_KC8, PQ_SRC_BITS8);
  if (ak == PQ_SRC_KC8 && bk == PQ_SRC_KC8) PQ_TILE_KINDS(true, PQ_SRC_KC8, PQ_SRC_KC8);
  if (ak == PQ_SRC_KC16 && bk == PQ_SRC_KC16) PQ_TILE_KINDS(false, PQ_SRC_KC16, PQ_SRC_KC16);
  if (ak == PQ_SRC_KC16 && bk == PQ_SRC_KS16) PQ_TILE_KINDS(false, PQ_SRC_KC16, PQ_SRC_KS16);
  if (ak == PQ_SRC_KC16 && bk == PQ_SRC_BITS16) PQ_TILE_KINDS(false, PQ_SRC_KC16, PQ_SRC_BITS16);
  if (ak == PQ_SRC_KS16 && bk == PQ_SRC_KS16) PQ_TILE_KINDS(false, PQ_SRC_KS16, PQ_SRC_KS16);
#undef PQ_TILE_KINDS
  return pq_set_error(PQ_ERR_BAD_ARG, "no MFMA kernel for operand kinds (%d, %d)", ak, bk);
}
