// Tiled MFMA GEMM for gfx950 with pluggable operand sources and epilogues.
//
//   C[m][n] (+)= epilogue( sum_k A(m,k) * B(n,k) )
//
// Operand sources (the 1-bit weights cross HBM and L2 as bits in every case: Sec. 3.1 W^INT1; App. A packing):
//   KC16 / KC8   contraction-contiguous rows, 16 bytes at a time;
//   KS16         contraction-strided sources (the transposed operands of the weight-gradient GEMMs);
//   BITS8/BITS16 packed sign bits, expanded to +/-1 (int8 or bf16).
// 256x256 tiles here, 128x256 where B is packed signs, smaller ones in pq_tile.hip.  The main loop sends operands from global memory straight into LDS: KC
// tiles as ROWS x 128 bytes, KS16 tiles as they lie in memory (read back with the transposing LDS read), and packed bits stay
// packed in LDS and are expanded in registers next to the MFMAs that consume them.  Contractions that are not whole steps
// fetch what is missing from a page of zeros.  The rank-r branch's second contraction rides in on the same ring.
// A wavefront owns a (BM/WGM) x (BN/WGN) sub-tile as 32x32 MFMA blocks:
//   v_mfma_f32_32x32x16_bf16 / v_mfma_i32_32x32x32_i8, 16 bytes of operand per lane per issue.
// LDS rows are 128 bytes with the 16-byte chunk index XOR-swizzled by the row so that the MFMA
// operand reads, the row-wise stores and the transposed stores are all free of bank conflicts.
#include <stdlib.h>
#include <string.h>
#include <type_traits>
#include "pq_epilogue.h"

#ifdef PQ_TRACE
// Instrumented builds only (never the shipped library): cycle stamps of two workgroups of the streaming loops, taken at
// points where no LDS read is outstanding (the stamp is a scalar-memory read and shares the counter LDS reads use).
__device__ unsigned long long pq_trace_buf[6][8][64][2];   // [3 kernel kinds x 2 workgroups][wave][step][before/after the barrier]
extern "C" int pq_debug_read_trace(unsigned long long* host_out) {
  return hipMemcpyFromSymbol(host_out, HIP_SYMBOL(pq_trace_buf), sizeof(unsigned long long) * 6 * 8 * 64 * 2) == hipSuccess ? 0 : -5;
}
#define PQ_STAMP(wg_slot, wave, step, which)                                                          \
  do {                                                                                                \
    if ((wg_slot) >= 0 && (step) < 64) {                                                              \
      const unsigned long long t_ = __builtin_readcyclecounter();                                     \
      if ((threadIdx.x & 63) == 0) pq_trace_buf[wg_slot][wave][step][which] = t_;                     \
    }                                                                                                 \
  } while (0)
#else
#define PQ_STAMP(wg_slot, wave, step, which) do { } while (0)
#endif

namespace {

[[maybe_unused]] __device__ __attribute__((aligned(256))) unsigned char pq_zero_page[256];   // never written

// Byte offset of 16-byte chunk c of row r in a tile whose rows are KB bytes (128 or 64).  The chunk
// index is XOR-swizzled by the row so that 8 consecutive rows at one logical chunk, and rows 8 apart
// at consecutive chunks (the transposing stores), fall into distinct 16-byte bank groups.
template <int KB>
__device__ __forceinline__ int lds_off(int r, int c) {
  if constexpr (KB == 128) return r * 128 + (((c ^ r ^ (r >> 3)) & 7) << 4);
  else return r * 64 + (((c ^ (r >> 1) ^ (r >> 3)) & 3) << 4);
}

// ---------------------------------------------------------------------------------------------
// Main loop: operands go from global memory straight into LDS
// (global_load_lds_dwordx4, no staging registers, no ds_write), and the contraction step is a fixed
// instruction order written as volatile asm statements: the fragment reads of MFMA group g+1 are issued
// before the MFMAs of group g, and the single barrier of a step sits before its last MFMA group, so the
// loads of the step after next and the first fragment reads of the next stage are issued under that
// group's MFMAs.  The compiler allocates the registers; the order of the statements is kept as written.
//   * contraction-contiguous operands (KC16, KC8): LDS tile [row][128 B], 16-byte chunks swizzled as
//     lds_off<128>; the swizzle is applied on the global side (lane l of a load instruction lands at LDS
//     byte 16 l of its 1 KB block, so it fetches the chunk that belongs there).
//   * contraction-strided operands (KS16): the tile stays as it is in memory, [64 contraction rows][512 B],
//     chunk c of row t stored at chunk c ^ 4 (t & 3); MFMA operands come from ds_read_b64_tr_b16, which
//     hands lane i of a 16-lane group element (i % 4) of the 8-byte row addressed by lane 4 e + i / 4,
//     e = 0..3: with lane j addressing (t = j / 4, 4 columns at 4 (j % 4)) lane i receives four consecutive
//     t of column i.
//   * packed-bit B operands stay packed in LDS (32-byte chunks of a row, two 16-byte direct loads per
//     wavefront and chunk, two chunk buffers) and are expanded to MFMA operands in registers, one dword
//     behind each MFMA; with B that small the A operand gets a ring of four stages instead of two.
//     Such a tile is 128x256 on four wavefronts, each with the 128x64 of the eight-wavefront tiles, and takes
//     exactly half of a CU's LDS: two workgroups that no barrier ties together share a CU, one multiplies while the
//     other starts, ends or waits, and a launch ends at half tiles.  Against 256x256 on eight wavefronts (same loop, 152 KB;
//     kernel times, us): 4096 rows 2048x2048 bf16 46.5 -> 35.9, 2048 rows 4096 -> 11008 int8 with r = 64 111.1 -> 98.7, 13032 rows
//     4096 -> 1472 bf16 184.6 -> 155.3, 8192 rows 2048x2048 59.6 -> 58.7; over 347 products 1.13 x, 0.93 x at worst (282
//     tiles: 26 CUs have two, the others one).  Where both fill the chip alike the matrix clock decides, which is the same.
// A wait on asm-issued reads names the registers it releases ("+v"), which orders their uses after it.
// ---------------------------------------------------------------------------------------------
#define PQ_DS_READ128(dst, addr, off) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(off) : "memory")
#define PQ_DS_READ64(dst, addr, off) asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(off) : "memory")
#define PQ_DS_READ_TR(dst, addr, off) asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(off) : "memory")
// The B fragment is passed as the first MFMA operand: the accumulator block is then the transpose of the usual
// one, lane l holds output row (l & 31) and register v holds column 8 (v >> 2) + 4 (l >> 5) + (v & 3), i.e. runs of
// four consecutive columns of one row, which the epilogue turns into 16-byte stores without going through LDS.
// Wave priority for the phases between two barriers of a streaming loop: 3, 2, 1, 0 from the phase after the barrier to the
// one before the next.  The two wavefronts of a SIMD then take turns: at equal priority the older one issues its group of
// MFMAs, which drops it below the other, and so on -- without it the older wavefront wins every arbitration, runs through
// its whole step and waits at the barrier while the younger one, alone on the SIMD, cannot hide its LDS latencies.
#define PQ_SETPRIO(n) asm volatile("s_setprio %0" ::"n"(n))
#define PQ_MFMA_BF16(acc, a, b) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %2, %1, %0" : "+v"(acc) : "v"(a), "v"(b))
#define PQ_MFMA_I8(acc, a, b) asm volatile("v_mfma_i32_32x32x32_i8 %0, %2, %1, %0" : "+v"(acc) : "v"(a), "v"(b))

// The result registers of an asm MFMA may be read by other instructions only when the matrix pipe has written them, up to 19
// issue slots later, and the compiler, which does not see an MFMA in the statement, puts no such distance there.  Whoever leaves
// a loop of asm MFMAs passes its accumulators through here: the waits, then a statement per accumulator that everything
// behind it depends on.  (A barrier in between hides the hazard by chance only: with four wavefronts to a workgroup the last
// register of the last block came out one product short.)
#define PQ_MFMA_SETTLE_FIRST() asm volatile("s_nop 15\n\ts_nop 3" ::: "memory")
template <typename ACC, int NB>
__device__ __forceinline__ void pq_mfma_settle(ACC (&acc)[NB]) {
#if defined(__HIP_DEVICE_COMPILE__)
  PQ_MFMA_SETTLE_FIRST();
#pragma unroll
  for (int j = 0; j < NB; ++j) asm volatile("" : "+v"(acc[j]));
#endif
}
template <typename ACC, int NA, int NB>
__device__ __forceinline__ void pq_mfma_settle(ACC (&acc)[NA][NB]) {
#if defined(__HIP_DEVICE_COMPILE__)
  PQ_MFMA_SETTLE_FIRST();
#pragma unroll
  for (int i = 0; i < NA; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) asm volatile("" : "+v"(acc[i][j]));
#endif
}

// One fragment set of a 128x64 wavefront tile: four A and two B operands of 16 bytes per lane.  Operands
// read with ds_read_b128 are whole (q), transposing reads deliver 8-byte halves (h) that the register
// allocator places next to each other.
template <bool ATR, bool BTR>
struct pq_frag_set {
  i32x4_t qa[ATR ? 1 : 4], qb[BTR ? 1 : 2];
  pq_i32x2 ha[ATR ? 8 : 1], hb[BTR ? 4 : 1];
  static constexpr int NREADS = (ATR ? 8 : 4) + (BTR ? 4 : 2);
  __device__ __forceinline__ i32x4_t A(int i) const {
    if constexpr (ATR) return i32x4_t{ha[2 * i][0], ha[2 * i][1], ha[2 * i + 1][0], ha[2 * i + 1][1]};
    else return qa[i];
  }
  __device__ __forceinline__ i32x4_t B(int j) const {
    if constexpr (BTR) return i32x4_t{hb[2 * j][0], hb[2 * j][1], hb[2 * j + 1][0], hb[2 * j + 1][1]};
    else return qb[j];
  }
  // waits until at most N_OUT LDS operations are outstanding; naming the registers orders their uses after it
  template <int N_OUT>
  __device__ __forceinline__ void wait() {
    if constexpr (!ATR && !BTR)
      asm volatile("s_waitcnt lgkmcnt(%6)" : "+v"(qa[0]), "+v"(qa[1]), "+v"(qa[2]), "+v"(qa[3]), "+v"(qb[0]), "+v"(qb[1]) : "n"(N_OUT));
    else if constexpr (ATR && BTR)
      asm volatile("s_waitcnt lgkmcnt(%12)"
                   : "+v"(ha[0]), "+v"(ha[1]), "+v"(ha[2]), "+v"(ha[3]), "+v"(ha[4]), "+v"(ha[5]), "+v"(ha[6]), "+v"(ha[7]),
                     "+v"(hb[0]), "+v"(hb[1]), "+v"(hb[2]), "+v"(hb[3])
                   : "n"(N_OUT));
    else if constexpr (ATR && !BTR)
      asm volatile("s_waitcnt lgkmcnt(%10)"
                   : "+v"(ha[0]), "+v"(ha[1]), "+v"(ha[2]), "+v"(ha[3]), "+v"(ha[4]), "+v"(ha[5]), "+v"(ha[6]), "+v"(ha[7]),
                     "+v"(qb[0]), "+v"(qb[1])
                   : "n"(N_OUT));
    else
      asm volatile("s_waitcnt lgkmcnt(%8)"
                   : "+v"(qa[0]), "+v"(qa[1]), "+v"(qa[2]), "+v"(qa[3]), "+v"(hb[0]), "+v"(hb[1]), "+v"(hb[2]), "+v"(hb[3])
                   : "n"(N_OUT));
  }
};

// ---------------------------------------------------------------------------------------------
// MFMA engine
// ---------------------------------------------------------------------------------------------
// One workgroup computes a BM x BN tile over the contraction range [z*kchunk, (z+1)*kchunk), z = blockIdx.y.
// DUAL: two problems of the same sizes (mode 3), blockIdx.z selects (an instantiation of its own: the test turns kernel
// arguments into run-time selections).  WHOLE: whole tiles (bf16 rows are stored without a look at the edges); TAIL: the contraction
// may end inside a step (an instantiation of its own: the registers its addresses take are spills elsewhere).  ACT: the product is the
// gradient of an FFN's hidden state (a plain bf16 output), which goes through the gated unit's derivative instead of to memory: `second`
// says where U and G are and dU and dG go.  The kernel waits for memory at its end only, and of two workgroups on a CU one multiplies
// meanwhile; in passes of its own the gradient was written and read once more (FFN of 8192 tokens 2048/5504, forward and backward:
// 1631 us with the gated unit apart, 1584 now).
template <int BM, int BN, int WGM, int WGN, int KB, bool WHOLE, bool TAIL, bool INT8, int AK, int BKIND, int AK2 = -1, int BK2 = -1, bool DUAL = false,
          bool ACT = false>
__global__ __launch_bounds__(WGM * WGN * 64, 2) void mfma_gemm_kernel(int M, int N, int K, pq_operand A,
                                                                     pq_operand B, pq_epilogue epi,
                                                                     int nbn, int total_tiles, int kchunk,
                                                                     float* splitk_part, pq_gemm_group grp,
                                                                     pq_phase2 ph2, typename std::conditional<ACT, pq_gemm_act, pq_second_arg<DUAL>>::type second) {
  constexpr int NT = WGM * WGN * 64;
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr int EPB = INT8 ? KB : KB / 2;  // contraction elements per LDS row
  constexpr int STAGE = (BM + BN) * KB;
  using acc_t = typename std::conditional<INT8, i32x16_t, f32x16_t>::type;

  // A packed-bit B operand stays packed in LDS (two buffers of 32 bytes per row), which leaves room for a ring of four stages
  // of the A operand: 80 KB with BM = 128, half of what a CU has, so the epilogue's few values lie where the bits were.
  constexpr bool BBITS = BKIND == PQ_SRC_BITS8 || BKIND == PQ_SRC_BITS16;
  constexpr int SMEM_BYTES = BBITS ? 4 * BM * KB + 2 * BN * 32 : 2 * STAGE;
  __shared__ __attribute__((aligned(16))) unsigned char smem[SMEM_BYTES + (BBITS ? 0 : 8 * (NT / 64) + 4 * BM)];
  unsigned char* const side = smem + (BBITS ? 4 * BM * KB : SMEM_BYTES);
  double* const red = (double*)side;
  float* const rowscale = (float*)(side + 8 * (NT / 64));   // per-row scale of the tile (one division per row, not per element)

  // XCD-aware tile order: consecutive workgroups go to different XCDs, so give each XCD a
  // contiguous range of tiles (its L2 then sees the same A row-panel for a run of tiles).
  // Work items are ordered (contraction split, tile row, tile column) and XCD c takes the c-th eighth of
  // that order: with a split contraction an XCD then works on one split and a band of tile rows, so the
  // operand panels it streams are shared by its workgroups instead of being fetched by every XCD.
  if constexpr (DUAL)
    if (blockIdx.z == 1) {                           // uniform
      A = second.A; B = second.B;
      epi.C = second.C; epi.dev_scale = second.dev_scale;
      splitk_part = second.part;
    }
  int pid = blockIdx.x, split = blockIdx.y;
  {
    const int nb = total_tiles * (int)gridDim.y;
    if ((nb & 7) == 0) {
      const int lin = blockIdx.x + total_tiles * blockIdx.y;
      const int w = (lin & 7) * (nb >> 3) + (lin >> 3);
      split = w / total_tiles;
      pid = w - split * total_tiles;
    }
  }
  const int bm = pid / nbn, bn = pid % nbn;
  int m0 = bm * BM;
  const int n0 = bn * BN;
  const int kb = split * kchunk;
  const int ke = min(K, kb + kchunk);
  const int Mtot = M;           // rows of C (a split's slab has Mtot rows)
  if (grp.mode == 1) {          // rows of group z: [offsets[z], offsets[z+1]); row tiles are numbered group after group
    int t = bm, z = 0;
    for (; z < grp.n_groups; ++z) {
      const int nt = (grp.offsets[z + 1] - grp.offsets[z] + BM - 1) / BM;
      if (t < nt) break;
      t -= nt;
    }
    if (z == grp.n_groups) return;   // uniform for the workgroup: the launch covers the worst-case tile count
    m0 = grp.offsets[z] + t * BM;
    M = grp.offsets[z + 1];
    B.p = (const char*)B.p + (size_t)z * grp.b_stride * (BKIND == PQ_SRC_KC8 ? 1 : 2);
    if (epi.col_div) epi.col_div += (size_t)z * grp.coldiv_stride;
  }

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave / WGN) * WM, wn0 = (wave % WGN) * WN;

  acc_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;

  const int nkt = ke > kb ? (ke - kb + EPB - 1) / EPB : 0;
  constexpr int NKS = KB / 32;   // MFMA issues along the contraction per LDS stage
  constexpr bool PH2 = (AK2 >= 0);
  static_assert(!PH2 || (BBITS && AK2 == PQ_SRC_KC16 && (BK2 == PQ_SRC_KC16 || BK2 == PQ_SRC_KS16)), "a second contraction rides in the ring of four");
  // A fused second contraction (K2 long, 64 to a step) comes in pieces of 16 KB, a ring stage each: 3 s: A2 of step s, 3 s + 1 and
  // 3 s + 2: the halves of its B2 (columns of a contraction-contiguous B2, contraction rows of a strided one).  Pieces 0 to 3 take
  // the ring's last four refills, which the main loop no longer needs, instead of being requested after it; piece j goes to
  // ring stage (nkt + j) mod 4.  Chunks past the end of K2 come from the page of zeros, in both operands.
  [[maybe_unused]] const int nk2 = PH2 ? (ph2.K2 + 63) >> 6 : 0;
  [[maybe_unused]] auto issue_ph2 = [&](int j, int stage) {
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (PH2) {
      const int s2 = j / 3, part = j - 3 * s2, k2 = s2 * 64;
      if (k2 >= ph2.K2) return;                      // uniform
      const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
      unsigned char* base = smem + stage * (BM * KB) + w * 4096;
      // the addresses are formed here, from opaque copies, so that nothing of them stays in registers across the main loop
      int ln = threadIdx.x & 63;
      asm volatile("" : "+v"(ln));
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int qi = w * 4 + i;
        const char* g;
        int pos;
        if (part == 0 || BK2 != PQ_SRC_KS16) {
          const pq_operand& op = part ? ph2.B2 : ph2.A2;
          const int row0 = part ? n0 + (part - 1) * 128 : m0, rows = part ? N : M;
          const int r = qi * 8 + (ln >> 3), pc = ln & 7;
          const int c = pc ^ ((r ^ (r >> 3)) & 7);
          const int grow = min(row0 + r, rows - 1);
          g = (const char*)op.p + ((size_t)grow * op.ld + k2) * 2 + c * 16;
          pos = k2 + c * 8;
        } else {
          const int t = (part - 1) * 32 + qi * 2 + (ln >> 5), pc = ln & 31;
          const int c = pc ^ (4 * (t & 3));
          int col = n0 + c * 8;
          if (col + 8 > N) col = n0;
          g = (const char*)ph2.B2.p + ((size_t)(k2 + t) * ph2.B2.ld + col) * 2;
          pos = k2 + t;
        }
        if (pos >= ph2.K2) g = (const char*)pq_zero_page;
        __builtin_amdgcn_global_load_lds(g, PQ_LDS_PTR(base + i * 1024), 16, 0, 0);
      }
    }
#endif
  };
  // per-thread LDS read offsets of the MFMA operand fragments (row part and swizzle part)
  int a_rb[TM], a_fx[TM], b_rb[TN], b_fx[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int r = wm0 + i * 32 + (lane & 31);
    a_rb[i] = lds_off<KB>(r, 0) & ~(KB - 1);
    a_fx[i] = (lds_off<KB>(r, 0) & (KB - 1)) >> 4;
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int r = wn0 + j * 32 + (lane & 31);
    b_rb[j] = BM * KB + (lds_off<KB>(r, 0) & ~(KB - 1));
    b_fx[j] = (lds_off<KB>(r, 0) & (KB - 1)) >> 4;
  }
  {
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass only needs the kernel's signature (LDS address-space casts are device-only)
    static_assert(BM == (BBITS ? 128 : 256) && BM == 128 * WGM && BN == 256 && WGN == 4 && KB == 128, "streaming loop: wavefront tiles of 128x64");
    constexpr bool ATR = (AK == PQ_SRC_KS16), BTR = (BKIND == PQ_SRC_KS16);
    constexpr bool BREG = BBITS;                      // B stays packed in LDS and is expanded per fragment
    constexpr int IPW = BREG ? 4 : 8;                 // 16-byte direct-load instructions per wavefront and stage
    constexpr int NSTAGE = BREG ? 4 : 2;              // depth of the LDS ring
    constexpr int STG = BREG ? BM * KB : STAGE;       // bytes per ring stage
    constexpr int RB = INT8 ? 16 : 8;                 // bytes of packed bits per B row and step
    constexpr int CH = 32 / RB;                       // steps covered by a 32-byte chunk of a packed row
    constexpr int BITS0 = NSTAGE * BM * KB;           // LDS offset of the two chunk buffers [256 rows][32 B]
    constexpr int AES = (AK == PQ_SRC_KC8) ? 1 : 2, BES = (BKIND == PQ_SRC_KC8) ? 1 : 2;
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    const uint32_t lds0 = (uint32_t)(size_t)smem;
#ifdef PQ_TRACE
    const int trace_kind = INT8 ? 0 : (BBITS ? 1 : 2);
    const int trace_slot = (blockIdx.y == 0 && blockIdx.z == 0 && (blockIdx.x == 0 || blockIdx.x == 100)) ? 2 * trace_kind + (blockIdx.x == 100) : -1;
#endif

    // ---- direct loads: instruction block qi of an operand is 1 KB of its LDS tile --------------------
    const bool opB = !BREG && wv >= 4;                // wave-uniform
    const int q0 = BREG ? wv * 4 : (wv & 3) * 8;
    const char* src[IPW];
    size_t adv;                                       // source bytes per contraction step
    {
      auto kc_src = [&](const pq_operand& op, int row0, int rows, int es, int qi) {
        const int r = qi * 8 + (lane >> 3), pc = lane & 7;
        const int c = pc ^ ((r ^ (r >> 3)) & 7);      // logical chunk stored at physical chunk pc of row r
        const int grow = min(row0 + r, rows - 1);      // rows past the end re-read the last row (never stored)
        return (const char*)op.p + ((size_t)grow * op.ld + kb) * es + c * 16;
      };
      auto ks_src = [&](const pq_operand& op, int col0, int cols, int qi) {
        const int t = qi * 2 + (lane >> 5), pc = lane & 31;
        const int c = pc ^ (4 * (t & 3));
        int col = col0 + c * 8;
        if (col + 8 > cols) col = col0;                // columns past the end: any valid chunk
        return (const char*)op.p + ((size_t)(kb + t) * op.ld + col) * 2;
      };
#pragma unroll
      for (int i = 0; i < IPW; ++i) {
        if (opB) {
          if constexpr (BTR) src[i] = ks_src(B, n0, N, q0 + i);
          else src[i] = kc_src(B, n0, N, BES, q0 + i);
        } else {
          if constexpr (ATR) src[i] = ks_src(A, m0, M, q0 + i);
          else src[i] = kc_src(A, m0, M, AES, q0 + i);
        }
      }
      if (opB) adv = BTR ? (size_t)64 * B.ld * 2 : (size_t)128;
      else adv = ATR ? (size_t)64 * A.ld * 2 : (size_t)128;
    }
    // A last step that the contraction does not fill takes its missing chunks (KC: 16 bytes of a row; KS16: a row) from a page
    // of zeros, in both operands; bits past the end may be anything then.
    auto issue = [&](int kt, int stage) {
      unsigned char* base = smem + stage * STG + (opB ? BM * KB : 0) + q0 * 1024;
      if (TAIL && (kt + 1) * EPB > ke - kb) {       // uniform
        const bool ks = opB ? BTR : ATR;
#pragma unroll
        for (int i = 0; i < IPW; ++i) {
          const int qi = q0 + i;
          const int pos = ks ? kt * EPB + qi * 2 + (lane >> 5) : kt * EPB + (((lane & 7) ^ ((lane >> 3) ^ qi)) & 7) * (EPB / 8);
          const char* g = pos < ke - kb ? src[i] + (size_t)kt * adv : (const char*)pq_zero_page;
          __builtin_amdgcn_global_load_lds(g, PQ_LDS_PTR(base + i * 1024), 16, 0, 0);
        }
        return;
      }
#pragma unroll
      for (int i = 0; i < IPW; ++i)
        __builtin_amdgcn_global_load_lds(src[i] + (size_t)kt * adv, PQ_LDS_PTR(base + i * 1024), 16, 0, 0);
    };
    // Packed bits of B: a row's bits are fetched 32 bytes (CH steps) at a time, two lanes per row, so a chunk
    // (256 rows, 8 KB) is one 16-byte load instruction per wavefront every CH steps.  Lanes 0..31 take the first
    // 16 bytes of the wavefront's 32 rows and lanes 32..63 the second, so in LDS a block of 32 rows is
    // [half][row][16 B]: the per-step reads (8 or 16 bytes of 32 consecutive rows) then walk consecutive
    // 16-byte slots instead of a 32-byte row stride (rows 8 apart on the same banks).
    // Rows that are not a multiple of 16 bytes (contractions that are not whole multiples of 128) are fetched a word per
    // lane, four loads per wavefront and chunk into the same places (the waits below then merely cover more loads of A).
    // What the last chunk lacks re-reads the start of the range into a place no step uses, or where A is zero.
    const int range_bytes = (ke - kb) >> 3;
    const bool words = TAIL && (B.ld & 15) != 0;     // uniform
    auto issue_bits = [&](int chunk, int buf) {
      constexpr int NB = 8 / (NT / 64);              // 32-row blocks per wavefront
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const int blk = wv * NB + u;
        unsigned char* dst = smem + BITS0 + buf * (BN * 32) + blk * 1024;
        if (words) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int row = min(n0 + blk * 32 + (i & 1) * 16 + (lane >> 2), N - 1);
            int off = chunk * 32 + (i >> 1) * 16 + (lane & 3) * 4;
            if (off + 4 > range_bytes) off = 0;
            const char* g = (const char*)B.p + (size_t)row * B.ld + (kb >> 3) + off;
            __builtin_amdgcn_global_load_lds(g, PQ_LDS_PTR(dst + i * 256), 4, 0, 0);
          }
          continue;
        }
        const int row = min(n0 + blk * 32 + (lane & 31), N - 1);
        int off = chunk * 32 + (lane >> 5) * 16;
        if (off + 16 > range_bytes) off = 0;
        const char* g = (const char*)B.p + (size_t)row * B.ld + (kb >> 3) + off;
        __builtin_amdgcn_global_load_lds(g, PQ_LDS_PTR(dst), 16, 0, 0);
      }
    };

    // ---- fragment read addresses (stage 0) ------------------------------------------------------------
    const int h = lane >> 5;
    uint32_t adA[ATR ? 4 : 8], adB[BTR ? 2 : 8];
    if constexpr (ATR) {
      const int tl = 8 * h + ((lane & 15) >> 2), cl = 16 * ((lane >> 4) & 1) + 4 * (lane & 3), sw = 4 * ((lane & 15) >> 2);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int col = wm0 + 32 * i + cl;
        adA[i] = lds0 + tl * 512 + (((col >> 3) ^ sw) << 4) + (col & 7) * 2;
      }
    } else {
#pragma unroll
      for (int pp = 0; pp < 2; ++pp)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) adA[pp * 4 + ks] = lds0 + a_rb[pp] + (((2 * ks + h) ^ a_fx[pp]) << 4);
    }
    if constexpr (BTR) {
      const int tl = 8 * h + ((lane & 15) >> 2), cl = 16 * ((lane >> 4) & 1) + 4 * (lane & 3), sw = 4 * ((lane & 15) >> 2);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int col = wn0 + 32 * j + cl;
        adB[j] = lds0 + BM * KB + tl * 512 + (((col >> 3) ^ sw) << 4) + (col & 7) * 2;
      }
    } else {
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) adB[j * 4 + ks] = lds0 + b_rb[j] + (((2 * ks + h) ^ b_fx[j]) << 4);
    }
    if constexpr (BREG) {
      // ---- ring of four stages: A streams as above, B stays packed ------------------------------------
      // A step's bits of a B row (8 or 16 bytes) are read once per wavefront tile column; the operand of
      // contraction sub-step s+1 is expanded from them in registers while the MFMAs of sub-step s issue,
      // one 4-byte piece behind each MFMA (a block of expansion instructions ahead of a block of MFMAs would
      // leave the matrix pipe idle for its length where the wavefronts of a SIMD run in step).
      // Every wavefront issues IPW direct loads of A per step, whatever the step (steps and chunks past the end
      // re-load the last one into a place nobody reads), plus its loads of bits, ahead of them, in the last
      // step of a chunk.  At the barrier of step t at most 2 IPW loads stay in flight, which leaves A up to
      // step t + 1 and the bits issued up to step t - 2 in LDS (when loads of bits are among the last 2 IPW,
      // the wait merely covers more loads of A).  Chunk c is issued behind the barrier of the last step of chunk
      // c - 2, from where on nobody reads that chunk, into its buffer, c mod 2; it is first read behind the
      // barrier of the last step of chunk c - 1, two steps later at least.
      static_assert(!ATR, "packed B goes with a contraction-contiguous A");
      using bits_t = typename std::conditional<INT8, i32x4_t, pq_i32x2>::type;
      struct aset {
        i32x4_t q[4];
        __device__ __forceinline__ void wait4() { asm volatile("s_waitcnt lgkmcnt(4)" : "+v"(q[0]), "+v"(q[1]), "+v"(q[2]), "+v"(q[3])); }
        __device__ __forceinline__ void wait0() { asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(q[0]), "+v"(q[1]), "+v"(q[2]), "+v"(q[3])); }
      };
      struct bfrag { int e[8]; };                      // two operands of four dwords
      aset G0, G1;
      bits_t bq0, bq1;
      const uint32_t adQ0 = lds0 + BITS0 + (wn0 / 32) * 1024 + (lane & 31) * 16, adQ1 = adQ0 + 1024;
      const uint32_t sh = INT8 ? 16u * h : 8u * h;
      // constants of the expansion kept in registers (three-operand encodings take no literals)
      uint32_t kM = INT8 ? 0x000001FFu : 0x80008000u, kC = 0x3F803F80u;
      asm volatile("" : "+v"(kM), "+v"(kC));
      auto read_a = [&](aset& G, auto ks_c, uint32_t so) {
        constexpr int ks = decltype(ks_c)::value;
        const uint32_t p0 = adA[ks] + so, p1 = adA[4 + ks] + so;
        PQ_DS_READ128(G.q[0], p0, 0);
        PQ_DS_READ128(G.q[1], p1, 0);
        PQ_DS_READ128(G.q[2], p0, 8192);
        PQ_DS_READ128(G.q[3], p1, 8192);
      };
      auto read_bits = [&](uint32_t so) {
        const uint32_t p0 = adQ0 + so, p1 = adQ1 + so;
        if constexpr (INT8) { PQ_DS_READ128(bq0, p0, 0); PQ_DS_READ128(bq1, p1, 0); }
        else { PQ_DS_READ64(bq0, p0, 0); PQ_DS_READ64(bq1, p1, 0); }
      };
      // bits of sub-step ks in the form the piecewise expansion takes: int8: the 16 bits; bf16: the 8
      // inverted bits at positions 0..7 and again at 15..22, so that one shift by 15 - 2d puts bits 2d
      // and 2d + 1 on the two sign positions of dword d
      auto prep = [&](const bits_t& q, auto ks_c) -> uint32_t {
        constexpr int ks = decltype(ks_c)::value;
        if constexpr (INT8) return (uint32_t)q[ks] >> sh;
        else {
          const uint32_t nb = ((((uint32_t)q[ks >> 1] >> (16 * (ks & 1))) >> sh) & 0xFFu) ^ 0xFFu;
          return nb | (nb << 15);
        }
      };
      // dword d of an operand: bf16: sign bits from the prepared word over the pattern (1.0, 1.0);
      // int8: nibble d -> one bit per byte (24-bit multiply) -> bytes 0x01 / 0xFF (byte permute)
#define PQ_EXPAND(dst, y, d)                                                                                     \
  do {                                                                                                           \
    if constexpr (INT8)                                                                                          \
      asm volatile("v_bfe_u32 %0, %1, %2, 4\n\tv_mul_u32_u24 %0, 0x204081, %0\n\tv_and_b32 %0, 0x1010101, %0\n\t" \
                   "v_perm_b32 %0, %3, %3, %0"                                                                    \
                   : "=&v"(dst)                                                                                  \
                   : "v"(y), "n"(4 * (d)), "v"(kM));                                                             \
    else                                                                                                         \
      asm volatile("v_lshlrev_b32 %0, %2, %1\n\tv_and_or_b32 %0, %0, %3, %4"                                      \
                   : "=&v"(dst)                                                                                  \
                   : "v"(y), "n"(15 - 2 * (d)), "v"(kM), "v"(kC));                                               \
  } while (0)
#define PQ_MFMA_AB(i, j, G, f0, f1)                                                          \
  do {                                                                                       \
    if constexpr (INT8) PQ_MFMA_I8(acc[i][j], G.q[i], (j) ? f1 : f0);                        \
    else PQ_MFMA_BF16(acc[i][j], G.q[i], (j) ? f1 : f0);                                     \
  } while (0)
      // MFMAs of one sub-step; FROM: the first MFMA that is followed by expansion pieces (0 = all eight)
      auto mfma_x = [&](const aset& G, const bfrag& cur, bfrag& nxt, uint32_t y0, uint32_t y1, auto from_c) {
        constexpr int FROM = decltype(from_c)::value;
        const i32x4_t f0 = {cur.e[0], cur.e[1], cur.e[2], cur.e[3]}, f1 = {cur.e[4], cur.e[5], cur.e[6], cur.e[7]};
        if constexpr (FROM == 0) {
          PQ_MFMA_AB(0, 0, G, f0, f1); PQ_EXPAND(nxt.e[0], y0, 0);
          PQ_MFMA_AB(0, 1, G, f0, f1); PQ_EXPAND(nxt.e[1], y0, 1);
          PQ_MFMA_AB(1, 0, G, f0, f1); PQ_EXPAND(nxt.e[2], y0, 2);
          PQ_MFMA_AB(1, 1, G, f0, f1); PQ_EXPAND(nxt.e[3], y0, 3);
          PQ_MFMA_AB(2, 0, G, f0, f1); PQ_EXPAND(nxt.e[4], y1, 0);
          PQ_MFMA_AB(2, 1, G, f0, f1); PQ_EXPAND(nxt.e[5], y1, 1);
          PQ_MFMA_AB(3, 0, G, f0, f1); PQ_EXPAND(nxt.e[6], y1, 2);
          PQ_MFMA_AB(3, 1, G, f0, f1); PQ_EXPAND(nxt.e[7], y1, 3);
        } else {
          PQ_MFMA_AB(1, 0, G, f0, f1); PQ_EXPAND(nxt.e[0], y0, 0); PQ_EXPAND(nxt.e[1], y0, 1);
          PQ_MFMA_AB(1, 1, G, f0, f1); PQ_EXPAND(nxt.e[2], y0, 2);
          PQ_MFMA_AB(2, 0, G, f0, f1); PQ_EXPAND(nxt.e[3], y0, 3); PQ_EXPAND(nxt.e[4], y1, 0);
          PQ_MFMA_AB(2, 1, G, f0, f1); PQ_EXPAND(nxt.e[5], y1, 1);
          PQ_MFMA_AB(3, 0, G, f0, f1); PQ_EXPAND(nxt.e[6], y1, 2);
          PQ_MFMA_AB(3, 1, G, f0, f1); PQ_EXPAND(nxt.e[7], y1, 3);
        }
      };
      using c0 = std::integral_constant<int, 0>;
      using c1 = std::integral_constant<int, 1>;
      using c2 = std::integral_constant<int, 2>;
      using c3 = std::integral_constant<int, 3>;
      bfrag fc, fn;
      const int nch = (nkt + CH - 1) / CH;              // the last chunk may be half used
      if (nkt > 0) {
        issue_bits(0, 0);
        issue_bits(min(1, nch - 1), 1);
#pragma unroll
        for (int s = 0; s < NSTAGE; ++s) issue(min(s, nkt - 1), s);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NSTAGE - 1) * IPW) : "memory");
        asm volatile("s_barrier" ::: "memory");
        read_bits(0u);
        read_a(G0, c0{}, 0u);
        asm volatile("s_waitcnt lgkmcnt(4)" : "+v"(bq0), "+v"(bq1));
        const uint32_t y0 = prep(bq0, c0{}), y1 = prep(bq1, c0{});
        PQ_EXPAND(fc.e[0], y0, 0); PQ_EXPAND(fc.e[1], y0, 1); PQ_EXPAND(fc.e[2], y0, 2); PQ_EXPAND(fc.e[3], y0, 3);
        PQ_EXPAND(fc.e[4], y1, 0); PQ_EXPAND(fc.e[5], y1, 1); PQ_EXPAND(fc.e[6], y1, 2); PQ_EXPAND(fc.e[7], y1, 3);
      }
      uint32_t so = 0u;
      int st = 0;
      int part = 0, buf = 0, chunk = 0;                 // position of the current step in the packed operand
      for (int kt = 0; kt < nkt; ++kt) {
        const int stn = (st + 1) & (NSTAGE - 1);
        const uint32_t sn = (uint32_t)stn * STG;
        const bool wrap = (part == CH - 1);
        const int partn = wrap ? 0 : part + 1;
        const int bufn = wrap ? buf ^ 1 : buf;
        PQ_SETPRIO(2);
        read_a(G1, c1{}, so);
        G0.wait4();
        mfma_x(G0, fc, fn, prep(bq0, c1{}), prep(bq1, c1{}), c0{});
        PQ_SETPRIO(1);
        read_a(G0, c2{}, so);
        G1.wait4();
        mfma_x(G1, fn, fc, prep(bq0, c2{}), prep(bq1, c2{}), c0{});
        PQ_SETPRIO(0);
        read_a(G1, c3{}, so);
        G0.wait4();
        mfma_x(G0, fc, fn, prep(bq0, c3{}), prep(bq1, c3{}), c0{});
        G1.wait0();                                     // every LDS read of this step is complete
        PQ_STAMP(trace_slot, wv, kt, 0);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * IPW) : "memory");
        asm volatile("s_barrier" ::: "memory");
        PQ_STAMP(trace_slot, wv, kt, 1);
        PQ_SETPRIO(3);
        if (wrap) issue_bits(min(chunk + 2, nch - 1), buf);   // everybody is done with this chunk
        // refill the stage just read: with the step four ahead, or, once there is none, with a piece of the second contraction
        if (PH2 && nk2 > 0 && nkt >= NSTAGE && kt + NSTAGE >= nkt) issue_ph2(kt + NSTAGE - nkt, st);
        else issue(min(kt + NSTAGE, nkt - 1), st);
        read_bits((uint32_t)(bufn * (BN * 32) + ((partn * RB) >> 4) * 512 + ((partn * RB) & 15)));   // past the last step: a place nobody uses
        read_a(G0, c0{}, sn);
        {
          const i32x4_t f0 = {fn.e[0], fn.e[1], fn.e[2], fn.e[3]}, f1 = {fn.e[4], fn.e[5], fn.e[6], fn.e[7]};
          PQ_MFMA_AB(0, 0, G1, f0, f1);
          PQ_MFMA_AB(0, 1, G1, f0, f1);
        }
        asm volatile("s_waitcnt lgkmcnt(4)" : "+v"(bq0), "+v"(bq1));   // the bits were requested ahead of G0's reads
        mfma_x(G1, fn, fc, prep(bq0, c0{}), prep(bq1, c0{}), c1{});
        st = stn;
        so = sn;
        part = partn;
        buf = bufn;
        chunk += wrap ? 1 : 0;
      }
      PQ_SETPRIO(0);
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
      pq_mfma_settle(acc);
#undef PQ_EXPAND
#undef PQ_MFMA_AB
    } else {
    using fset = pq_frag_set<ATR, BTR>;
    fset F0, F1;
    auto read_set = [&](fset& F, auto ks_c, uint32_t so) {
      constexpr int ks = decltype(ks_c)::value;
      if constexpr (ATR) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t pa = adA[i] + so;
          PQ_DS_READ_TR(F.ha[2 * i], pa, ks * 8192);
          PQ_DS_READ_TR(F.ha[2 * i + 1], pa, ks * 8192 + 2048);
        }
      } else {
        const uint32_t p0 = adA[ks] + so, p1 = adA[4 + ks] + so;
        PQ_DS_READ128(F.qa[0], p0, 0);
        PQ_DS_READ128(F.qa[1], p1, 0);
        PQ_DS_READ128(F.qa[2], p0, 8192);
        PQ_DS_READ128(F.qa[3], p1, 8192);
      }
      if constexpr (BTR) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const uint32_t pb = adB[j] + so;
          PQ_DS_READ_TR(F.hb[2 * j], pb, ks * 8192);
          PQ_DS_READ_TR(F.hb[2 * j + 1], pb, ks * 8192 + 2048);
        }
      } else {
        const uint32_t pb0 = adB[ks] + so, pb1 = adB[4 + ks] + so;
        PQ_DS_READ128(F.qb[0], pb0, 0);
        PQ_DS_READ128(F.qb[1], pb1, 0);
      }
    };
    auto mfma_set = [&](const fset& F) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const i32x4_t fa = F.A(i);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const i32x4_t fb = F.B(j);
          if constexpr (INT8) PQ_MFMA_I8(acc[i][j], fa, fb);
          else PQ_MFMA_BF16(acc[i][j], fa, fb);
        }
      }
    };
    using c0 = std::integral_constant<int, 0>;
    using c1 = std::integral_constant<int, 1>;
    using c2 = std::integral_constant<int, 2>;
    using c3 = std::integral_constant<int, 3>;
    constexpr int NR = fset::NREADS;

    if (nkt > 0) {
      issue(0, 0);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      asm volatile("s_barrier" ::: "memory");
      if (nkt > 1) issue(1, 1);
      read_set(F0, c0{}, 0u);
    }
    for (int kt = 0; kt < nkt; ++kt) {
      const uint32_t so = (kt & 1) ? (uint32_t)STAGE : 0u, sn = (kt & 1) ? 0u : (uint32_t)STAGE;
      PQ_SETPRIO(2);
      read_set(F1, c1{}, so);
      F0.template wait<NR>();
      mfma_set(F0);
      PQ_SETPRIO(1);
      read_set(F0, c2{}, so);
      F1.template wait<NR>();
      mfma_set(F1);
      PQ_SETPRIO(0);
      read_set(F1, c3{}, so);
      F0.template wait<NR>();
      mfma_set(F0);
      F1.template wait<0>();                          // every LDS access of this step is complete
      PQ_STAMP(trace_slot, wv, kt, 0);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the direct loads of the next stage have landed
      asm volatile("s_barrier" ::: "memory");
      PQ_STAMP(trace_slot, wv, kt, 1);
      PQ_SETPRIO(3);
      if (kt + 2 < nkt) issue(kt + 2, kt & 1);
      if (kt + 1 < nkt) read_set(F0, c0{}, sn);
      mfma_set(F1);
    }
    PQ_SETPRIO(0);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    pq_mfma_settle(acc);
    }
#endif
  }
  __syncthreads();  // all MFMA operand reads are done: LDS is reused below

  // Optional second contraction (rank-r branch): rescale the first accumulator, then a short bf16 loop over K2 into the same
  // tile.  The pieces of its first step (and A2 of the second) already sit in the ring; what a third and later steps need is
  // requested when the one before has been read, and the other workgroup of the CU has the matrix pipe meanwhile.
  constexpr bool ACC_INT = INT8 && !PH2;
  f32x16_t accf[PH2 ? TM : 1][PH2 ? TN : 1];
  if constexpr (PH2) {
#if defined(__HIP_DEVICE_COMPILE__)
    typedef short v4s_t __attribute__((ext_vector_type(4)));
    if (nkt < 4) {                                   // uniform: the loop had no refills to spare
#pragma unroll
      for (int j = 0; j < 4; ++j) issue_ph2(j, (nkt + j) & 3);
    }
    const float sc1 = ph2.dev_scale1 ? __fmul_rn(ph2.scale1, *ph2.dev_scale1) : ph2.scale1;
    if (ph2.row_div1) {                              // uniform: one divisor load and one division per row of the tile
      for (int r = tid; r < BM; r += NT) rowscale[r] = sc1 / ph2.row_div1[min(m0 + r, M - 1)];
      __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const float sr = ph2.row_div1 ? rowscale[wm0 + i * 32 + (lane & 31)] : sc1;   // a lane holds one row of a block
#pragma unroll
      for (int v = 0; v < 16; ++v)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const auto e1 = acc[i][j][v];
          accf[i][j][v] = (float)e1 * sr;
        }
    }
    const int hh = lane >> 5;
    auto piece = [&](int j) { return smem + ((nkt + j) & 3) * (BM * KB); };
    for (int s2 = 0; s2 < nk2; ++s2) {
      if (s2 > 0) {
        // both halves of this step's B2, and the next one's A2 where that of the step before was
        __syncthreads();
        issue_ph2(3 * s2 + 1, (nkt + 1) & 3);
        issue_ph2(3 * s2 + 2, (nkt + 2) & 3);
        if (s2 + 1 < nk2) issue_ph2(3 * s2 + 3, (nkt + (s2 & 1 ? 0 : 3)) & 3);
      }
      if (s2 > 0 || nkt < 4) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
      }
      const unsigned char* ta = piece(s2 & 1 ? 3 : 0);
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        const int ch = 2 * ks + hh;
        uint4 fa[TM], fb[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[i] = *reinterpret_cast<const uint4*>(ta + a_rb[i] + ((ch ^ a_fx[i]) << 4));
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          if constexpr (BK2 == PQ_SRC_KS16) {
            // [64 contraction rows][256 columns] as it lies in memory, 16-byte chunks of a row swizzled by the row:
            // two transposing reads (rows 16 ks + 8 h + (0..3), then + 4) make the operand of 8 contraction indices
            const int tl = 8 * hh + ((lane & 15) >> 2), cl = 16 * ((lane >> 4) & 1) + 4 * (lane & 3), sw = 4 * ((lane & 15) >> 2);
            const int col = wn0 + 32 * j + cl;
            const unsigned char* pb = piece(1 + (ks >> 1)) + (ks & 1) * 8192 + tl * 512 + (((col >> 3) ^ sw) << 4) + (col & 7) * 2;
            const v4s_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s_t*)(pb));
            const v4s_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s_t*)(pb + 2048));
            const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
            fb[j] = make_uint4(l2.x, l2.y, h2.x, h2.y);
          } else {
            // [256 columns][128 B], 128 columns to a piece
            const int r = (wn0 & 127) + 32 * j + (lane & 31), o = lds_off<KB>(r, 0);
            fb[j] = *reinterpret_cast<const uint4*>(piece(1 + (wn0 >> 7)) + (o & ~(KB - 1)) + ((ch ^ ((o & (KB - 1)) >> 4)) << 4));
          }
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            accf[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, fb[j]), __builtin_bit_cast(bf16x8_t, fa[i]),
                                                                 accf[i][j], 0, 0, 0);
      }
    }
#endif
    __syncthreads();
  }
  // Epilogue: in a 32x32 accumulator block lane l holds row (l & 31) and, per group g = v >> 2, the four columns
  // 8 g + 4 (l >> 5) + (0..3).  One half-wave exchange per register (v_permlane32_swap: the upper half of the first
  // operand against the lower half of the second) gives the lower lanes the eight columns of the even groups and
  // the upper lanes those of the odd groups, so every lane stores 8 consecutive columns of its row at a time
  // (two neighbouring lanes = 16 consecutive columns) and nothing passes through LDS.  With a split contraction
  // the raw fp32 accumulators go to this split's slab instead; splitk_reduce_kernel finishes the job.
  epi_state st;
  epi_begin(epi, st);
  float* slab = splitk_part ? splitk_part + (size_t)split * Mtot * N : nullptr;
  const bool row_scaled = !slab && epi.row_div != nullptr;   // uniform
  if (row_scaled) {
    for (int r = tid; r < BM; r += NT) rowscale[r] = st.sc0 / epi.row_div[min(m0 + r, M - 1)];
    __syncthreads();
  }
#ifdef PQ_NO_STAGE
  constexpr bool CAN_STAGE = false;
#else
  constexpr bool CAN_STAGE = SMEM_BYTES >= (NT / 64) * 16384;
#endif
  // (store limits: fp32 outputs only, where a 16-byte chunk is four columns and the column limit a multiple of four)
  const bool raw = slab || epi.out_kind == PQ_OUT_I32;       // uniform: the accumulators as they are
  const bool staged = CAN_STAGE && (slab || (epi.out_kind == PQ_OUT_I32 && epi.m_limit == 0 && epi.n_limit == 0) || ((epi.out_kind == PQ_OUT_F32 || (epi.out_kind == PQ_OUT_BF16 && epi.m_limit == 0 && epi.n_limit == 0)) &&
                                             !epi.col_div && !epi.maskW && !epi.accumulate && !epi.dot_comp &&
                                             !epi.sign_bytes));   // uniform
  if (staged) {
    const bool o16 = !slab && epi.out_kind == PQ_OUT_BF16;
    int tid_e = threadIdx.x;
    asm volatile("" : "+v"(tid_e));
    const int lane_e = tid_e & 63, wave_e = tid_e >> 6;
    const int wm0_e = (wave_e / WGN) * WM, wn0_e = (wave_e % WGN) * WN;
    unsigned char* wreg = smem + wave_e * 16384;
    char* outp = slab ? (char*)slab : (char*)epi.C;
    const size_t ldo = slab ? (size_t)N * 4 : (size_t)epi.ldc * (o16 ? 2 : 4);
    const int hh = lane_e >> 5;
    const int mlim = (!slab && epi.m_limit > 0 && epi.m_limit < M) ? epi.m_limit : M;
    const int nlim = (!slab && epi.n_limit > 0 && epi.n_limit < N) ? epi.n_limit : N;
    const pq_gemm_act act = [&] {
      if constexpr (ACT) return second;
      else return pq_gemm_act{};
    }();
    auto run = [&](auto o16_c) {
    constexpr bool o16 = decltype(o16_c)::value;
#pragma unroll
    for (int pass = 0; pass < (o16 ? 1 : 2); ++pass) {
#pragma unroll
      for (int ii = 0; ii < (o16 ? TM : TM / 2); ++ii) {
        const int i = o16 ? ii : pass * (TM / 2) + ii;
        const int rl = ii * 32 + (lane_e & 31);
        const int m = m0 + wm0_e + i * 32 + (lane_e & 31);
        const float rs = row_scaled ? rowscale[m - m0] : __builtin_nanf("");
#pragma unroll
        for (int j = 0; j < TN; ++j) {
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            uint32_t w[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              if (raw) {
                // copy the element out first: a vector element is not a bit_cast-able lvalue
                if constexpr (PH2) { const float e = accf[i][j][4 * g + t]; w[t] = __float_as_uint(e); }
                else { const auto e = acc[i][j][4 * g + t]; w[t] = __builtin_bit_cast(uint32_t, e); }
              } else {
                const float sc = row_scaled ? rs : st.sc0;
                float a;
                if constexpr (PH2) a = accf[i][j][4 * g + t];
                else a = (float)acc[i][j][4 * g + t];
                w[t] = __float_as_uint(__fmul_rn(sc, a));
              }
            }
            if constexpr (o16) {
              const uint2 o = make_uint2(pack_bf16x2(__uint_as_float(w[0]), __uint_as_float(w[1])),
                                         pack_bf16x2(__uint_as_float(w[2]), __uint_as_float(w[3])));
              *reinterpret_cast<uint2*>(wreg + rl * 128 + (((j * 4 + g) ^ (rl & 7)) << 4) + hh * 8) = o;
            } else {
              // written as asm with two wait states behind it: the compiler puts no distance between a 16-byte LDS store and a
              // VALU write to its data registers (it does for 16-byte global stores), and a staged epilogue whose last store was
              // followed at once by such writes lost that store's data in part
              const i32x4_t o = {(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
              const uint32_t ad = (uint32_t)(size_t)(wreg + rl * 256 + (((j * 8 + 2 * g + hh) ^ (rl & 7)) << 4));
              asm volatile("ds_write_b128 %0, %1\n\ts_nop 1" ::"v"(ad), "v"(o) : "memory");
            }
          }
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_wave_barrier();
      if constexpr (o16 && ACT) {
#pragma unroll
        for (int ib = 0; ib < 16; ib += 4) {           // four rows' U and G requested together (clamped: edge rows are not stored)
          uint4 u[4], g[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int m = min(m0 + wm0_e + (ib + q) * 8 + (lane_e >> 3), M - 1), n = min(n0 + wn0_e + (lane_e & 7) * 8, N - 8);
            u[q] = *reinterpret_cast<const uint4*>((const uint16_t*)act.U + (size_t)m * N + n);
            g[q] = *reinterpret_cast<const uint4*>((const uint16_t*)act.G + (size_t)m * N + n);
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int rl = (ib + q) * 8 + (lane_e >> 3), c = lane_e & 7;
            const uint4 v = *reinterpret_cast<const uint4*>(wreg + rl * 128 + ((c ^ (rl & 7)) << 4));
            const int m = m0 + wm0_e + rl, n = n0 + wn0_e + c * 8;
            uint4 du, dg;
            pq_swiglu_bwd8(v, u[q], g[q], n, act.Fv, du, dg);
            if (m < M && n < N) {
              *reinterpret_cast<uint4*>((uint16_t*)act.dU + (size_t)m * N + n) = du;
              *reinterpret_cast<uint4*>((uint16_t*)act.dG + (size_t)m * N + n) = dg;
            }
          }
        }
      } else if constexpr (o16) {
#pragma unroll
        for (int it = 0; it < 16; ++it) {
          const int rl = it * 8 + (lane_e >> 3), c = lane_e & 7;
          const uint4 v = *reinterpret_cast<const uint4*>(wreg + rl * 128 + ((c ^ (rl & 7)) << 4));
          const int m = m0 + wm0_e + rl, n = n0 + wn0_e + c * 8;
          if (WHOLE || (m < M && n < N)) *reinterpret_cast<uint4*>(outp + (size_t)m * ldo + (size_t)n * 2) = v;
        }
      } else {
#pragma unroll
        for (int it = 0; it < 16; ++it) {
          const int rl = it * 4 + (lane_e >> 4), c = lane_e & 15;
          const uint4 v = *reinterpret_cast<const uint4*>(wreg + rl * 256 + ((c ^ (rl & 7)) << 4));
          const int m = m0 + wm0_e + pass * 64 + rl, n = n0 + wn0_e + c * 4;
          if (m < mlim && n < nlim) *reinterpret_cast<uint4*>(outp + (size_t)m * ldo + (size_t)n * 4) = v;
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_wave_barrier();
    }
    };
    if (o16) run(std::true_type{});
    else run(std::false_type{});
    if (!slab) epi_end<NT>(epi, st, red, blockIdx.x);
    return;
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m0 + wm0 + i * 32 + (lane & 31);
    const float rs = row_scaled ? rowscale[m - m0] : __builtin_nanf("");
#pragma unroll
    for (int j = 0; j < TN; ++j) {
#pragma unroll
      for (int pr = 0; pr < 2; ++pr) {
        uint32_t x[4], y[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          uint32_t lo, hi;
          // copy the elements out first: a vector element is not a bit_cast-able lvalue
          if constexpr (PH2) {
            const float e0 = accf[i][j][8 * pr + t], e1 = accf[i][j][8 * pr + 4 + t];
            lo = __builtin_bit_cast(uint32_t, e0); hi = __builtin_bit_cast(uint32_t, e1);
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
            epi_vec8<ACC_INT, BKIND == PQ_SRC_KC8>(epi, st, m, n, r0, r1, rs);
          }
        }
      }
    }
  }
  if (!slab) epi_end<NT>(epi, st, red, blockIdx.x);
}

// Second stage of a split contraction: sum the slabs in index order (deterministic), then apply
// the caller's epilogue.  One thread per 8 consecutive columns.
// INT: the slabs hold int32 accumulators (int8 engine); their sum is exact.
template <bool INT, bool TWO>
__device__ __forceinline__ void splitk_reduce_body(int M, int N, int splits, const float* __restrict__ part, const pq_epilogue& epi,
                                                   int block) {
  __shared__ double red[4];
  const size_t n8 = (size_t)N / 8, total = (size_t)M * n8;
  const size_t idx = (size_t)block * 256 + threadIdx.x;
  epi_state st;
  epi_begin(epi, st);
  if (idx < total) {
    const int m = (int)(idx / n8), n = (int)(idx % n8) * 8;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
    int4 ia = make_int4(0, 0, 0, 0), ib = ia;
    const size_t slab = (size_t)M * N;
    // four slabs are requested together (slabs past the end repeat the last one and are dropped): a load behind
    // a loop-carried wait would cost one memory latency per slab; the sums still run in slab order
    for (int z = 0; z < splits; z += 4) {
      float4 x[4], y[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float* p = part + (size_t)min(z + u, splits - 1) * slab + (size_t)m * N + n;
        x[u] = *reinterpret_cast<const float4*>(p);
        y[u] = *reinterpret_cast<const float4*>(p + 4);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (z + u < splits) {
          if constexpr (INT) {
            ia.x += __float_as_int(x[u].x); ia.y += __float_as_int(x[u].y); ia.z += __float_as_int(x[u].z); ia.w += __float_as_int(x[u].w);
            ib.x += __float_as_int(y[u].x); ib.y += __float_as_int(y[u].y); ib.z += __float_as_int(y[u].z); ib.w += __float_as_int(y[u].w);
          } else {
            a.x += x[u].x; a.y += x[u].y; a.z += x[u].z; a.w += x[u].w;
            b.x += y[u].x; b.y += y[u].y; b.z += y[u].z; b.w += y[u].w;
          }
        }
    }
    if constexpr (INT) {
      epi_vec8<true>(epi, st, m, n, make_uint4((uint32_t)ia.x, (uint32_t)ia.y, (uint32_t)ia.z, (uint32_t)ia.w),
                     make_uint4((uint32_t)ib.x, (uint32_t)ib.y, (uint32_t)ib.z, (uint32_t)ib.w));
    } else {
      const uint4 r0 = make_uint4(__float_as_uint(a.x), __float_as_uint(a.y), __float_as_uint(a.z), __float_as_uint(a.w));
      const uint4 r1 = make_uint4(__float_as_uint(b.x), __float_as_uint(b.y), __float_as_uint(b.z), __float_as_uint(b.w));
      epi_vec8<false, TWO>(epi, st, m, n, r0, r1);
    }
  }
  epi_end<256>(epi, st, red, block);
}

template <bool INT, bool TWO>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(int M, int N, int splits, const float* __restrict__ part,
                                                            pq_epilogue epi) {
  splitk_reduce_body<INT, TWO>(M, N, splits, part, epi, blockIdx.x);
}

// The reductions of a paired launch in one launch: the first nblk0 workgroups finish problem 0, the rest problem 1.
// Up to two scalar reductions of the same call (d alpha, d beta) ride along as the last workgroups of the grid.
template <bool INT>
__global__ __launch_bounds__(256) void splitk_reduce_pair_kernel(int splits, int nblk0, int nblk1, int M0, int N0,
                                                                 const float* __restrict__ part0, pq_epilogue epi0, int M1, int N1,
                                                                 const float* __restrict__ part1, pq_epilogue epi1, pq_reduce_job j0,
                                                                 pq_reduce_job j1) {
  const int b = blockIdx.x;
  if (b < nblk0) splitk_reduce_body<INT, false>(M0, N0, splits, part0, epi0, b);
  else if (b < nblk0 + nblk1) splitk_reduce_body<INT, false>(M1, N1, splits, part1, epi1, b - nblk0);
  else pq_reduce_job_body(b == nblk0 + nblk1 ? j0 : j1);
}

// ---------------------------------------------------------------------------------------------
// Weight-gradient GEMMs (both operands bf16 with the contraction index as rows: dW = dY^T X over the tokens):
// a 256x256 or 192x256 tile on FOUR wavefronts.
// ---------------------------------------------------------------------------------------------
// With real (non-constant) operand data the chip runs these kernels against its power limit: the shader clock of the
// eight-wavefront kernel above falls from 2.3 GHz on all-zero operands to 1.7 GHz on normally distributed ones, and what
// LDS reads and direct loads cost shows as clock, not as stalls.  A wavefront that owns 128x128 of the tile reads eight
// operand blocks per sixteen MFMAs where a 128x64 one reads six per eight: a third less LDS traffic for the same products.
// Its 256 accumulator registers live in AGPRs (one wavefront per SIMD has 512 registers), which leaves the arch VGPRs for
// two fragment sets.  One wavefront per SIMD keeps the matrix pipe busy on its own as long as every wait it meets has
// been satisfied long before, so the order below is fixed (volatile asm statements): a stage is 32 contraction rows
// ([32][512 B] per operand, chunk c of row t at chunk c ^ 4 (t & 3), as in the streaming loop above), the ring has four
// stages, and per stage a wavefront issues 32 MFMAs in four groups of eight: behind each MFMA of groups 0 and 2 goes one
// operand block (two transposing reads) of the fragment set after the current one, behind each MFMA of group 1 one direct
// load of the stage three ahead.  The single barrier of a stage sits between groups 0 and 1: by then the wavefront's own
// loads of the next stage have landed (vmcnt), after it everybody's have and nobody reads the stage before the current
// one, whose slot the new loads take.  Past the last stage the loads re-request the last one into a free slot, so the
// counters stay uniform.
// With 192 rows to a tile a wavefront has three blocks of A instead of four, i.e. 24 MFMAs to fourteen reads of operand blocks
// (32 to sixteen) and 28 KB of loads a stage: 0.86 of a 256x256 stage for 0.75 of its products, worth it where the larger tile
// leaves CUs idle (5504x2048: 176 tiles, or 232).  A's contraction rows are 384 bytes then, chunk c of row t at c ^ 4 (t >> 1 & 1).
// The epilogue passes the accumulators through the wavefront's 32 KB of the ring, 64 rows at a time, and reads whole
// 512-byte rows back: raw slabs of a split contraction and plain fp32 outputs leave as 16-byte stores of whole rows, every
// other epilogue goes through epi_vec8 with eight consecutive columns per lane.
#define PQ_MFMA_BF16_ACC(acc, a, b) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %2, %1, %0" : "+a"(acc) : "v"(a), "v"(b))
template <int TA>
struct pq_frag_set_w4 {
  pq_i32x2 h[2 * TA + 8];   // h[2q], h[2q+1]: the halves of operand block q; q < TA rows of A (tile rows), then four of B (tile columns)
  __device__ __forceinline__ i32x4_t op(int q) const { return i32x4_t{h[2 * q][0], h[2 * q][1], h[2 * q + 1][0], h[2 * q + 1][1]}; }
  __device__ __forceinline__ void wait_all() {
    if constexpr (TA == 3)
      asm volatile("s_waitcnt lgkmcnt(0)"
                   : "+v"(h[0]), "+v"(h[1]), "+v"(h[2]), "+v"(h[3]), "+v"(h[4]), "+v"(h[5]), "+v"(h[6]), "+v"(h[7]), "+v"(h[8]), "+v"(h[9]),
                     "+v"(h[10]), "+v"(h[11]), "+v"(h[12]), "+v"(h[13]));
    else
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(h[0]), "+v"(h[1]), "+v"(h[2]), "+v"(h[3]), "+v"(h[4]), "+v"(h[5]), "+v"(h[6]), "+v"(h[7]), "+v"(h[8]), "+v"(h[9]),
                   "+v"(h[10]), "+v"(h[11]), "+v"(h[12]), "+v"(h[13]), "+v"(h[14]), "+v"(h[15]));
  }
};

// RAGGED: the last stage of a range is not whole; its missing rows come from a page of zeros.  (An instantiation of its own: the
// test behind every load cost the whole ones 3 to 4 %.)  TWO: the epilogue has a second destination.  TA: 32-row blocks of A that a
// wavefront multiplies, 4 (256x256 tiles) or 3 (192x256).
template <int TA, bool RAGGED, bool DUAL, bool TWO>
__device__ __forceinline__ void gemm_tn_w4_body(int M, int N, int K, pq_operand A, pq_operand B, pq_epilogue epi, int nbn,
                                                int total_tiles, int kchunk, float* splitk_part, pq_second_arg<DUAL> second) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int BM = 64 * TA, RSA = 2 * BM;          // tile rows; bytes of a contraction row of A in LDS
  constexpr int IPS = TA + 4;                        // load instructions per wavefront and stage
  constexpr int NM = 4 * TA;                         // MFMAs per wavefront and half stage
  // chunk c of contraction row t lies at c ^ swzA(t), four rows of 32 columns on distinct banks whatever the row length
  auto swzA = [](int t) { return TA == 4 ? 4 * (t & 3) : 4 * ((t >> 1) & 1); };
  constexpr int STG = 32768;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[4 * STG];
  __shared__ double red[4];
  if constexpr (DUAL)
    if (blockIdx.z == 1) {                           // uniform: the second of two problems of the same sizes
      A = second.A; B = second.B; epi.C = second.C; epi.dev_scale = second.dev_scale;
      splitk_part = second.part;
    }
  int pid = blockIdx.x, split = blockIdx.y;
  {   // XCD-aware order, as in mfma_gemm_kernel
    const int nb = total_tiles * (int)gridDim.y;
    if ((nb & 7) == 0) {
      const int lin = blockIdx.x + total_tiles * blockIdx.y;
      const int w = (lin & 7) * (nb >> 3) + (lin >> 3);
      split = w / total_tiles;
      pid = w - split * total_tiles;
    }
  }
  const int bm = pid / nbn, bn = pid % nbn;
  const int m0 = bm * BM, n0 = bn * 256;
  const int kb = split * kchunk, ke = min(K, kb + kchunk);
  const int nkt = ke > kb ? (ke - kb + (RAGGED ? 31 : 0)) >> 5 : 0;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm0 = (wv >> 1) * 32 * TA, wn0 = (wv & 1) * 128;
  const uint32_t lds0 = (uint32_t)(size_t)smem;

  // direct loads: instruction block qi of an operand is 1 KB of its stage (of B: two contraction rows); a wavefront owns TA
  // blocks of A and four of B.  Columns past the end fetch the tile's first chunk (any valid address: never stored).
  const char* src[IPS];
  int trow[IPS];
#pragma unroll
  for (int i = 0; i < IPS; ++i) {
    const bool isA = i < TA;
    const int l = (isA ? wv * TA + i : wv * 4 + i - TA) * 64 + lane, cpr = isA ? 8 * TA : 32;
    const int t = l / cpr, pc = l - t * cpr;
    const int c = pc ^ (isA ? swzA(t) : 4 * (t & 3));
    const pq_operand& op = isA ? A : B;
    const int col0 = isA ? m0 : n0, cols = isA ? M : N;
    trow[i] = t;
    int col = col0 + c * 8;
    if (col + 8 > cols) col = col0;
    src[i] = (const char*)op.p + ((size_t)(kb + t) * op.ld + col) * 2;
  }
  const size_t advA = (size_t)32 * A.ld * 2, advB = (size_t)32 * B.ld * 2;
  auto issue1 = [&](int kt, int slot, int i) {
    unsigned char* dst = smem + slot * STG + (i < TA ? (wv * TA + i) * 1024 : 16384 + (wv * 4 + i - TA) * 1024);
    const char* g = src[i] + (size_t)kt * (i < TA ? advA : advB);
    if (RAGGED && kt == nkt - 1 && kt * 32 + trow[i] >= ke - kb) g = (const char*)pq_zero_page;
    __builtin_amdgcn_global_load_lds(g, PQ_LDS_PTR(dst), 16, 0, 0);
  };

  // fragment read addresses (slot 0, contraction rows 0..15): see the transposing reads of the streaming loop
  uint32_t ad[IPS];
  {
    const int h = lane >> 5;
    const int tl = 8 * h + ((lane & 15) >> 2), cl = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
#pragma unroll
    for (int q = 0; q < IPS; ++q) {
      const int col = (q < TA ? wm0 + 32 * q : wn0 + 32 * (q - TA)) + cl;
      ad[q] = lds0 + (q < TA ? tl * RSA : 16384 + tl * 512) + (((col >> 3) ^ (q < TA ? swzA(tl) : 4 * (tl & 3))) << 4) + (col & 7) * 2;
    }
  }
  using fset = pq_frag_set_w4<TA>;
  fset F0, F1;
  auto rd = [&](fset& F, int q, uint32_t so, auto ks_c) {
    constexpr int ks = decltype(ks_c)::value;
    const uint32_t pa = ad[q] + so;
    if (q < TA) {                                    // (constant after unrolling)
      PQ_DS_READ_TR(F.h[2 * q], pa, ks * 16 * RSA);
      PQ_DS_READ_TR(F.h[2 * q + 1], pa, ks * 16 * RSA + 4 * RSA);
    } else {
      PQ_DS_READ_TR(F.h[2 * q], pa, ks * 8192);
      PQ_DS_READ_TR(F.h[2 * q + 1], pa, ks * 8192 + 2048);
    }
  };
  using c0 = std::integral_constant<int, 0>;
  using c1 = std::integral_constant<int, 1>;

  if (nkt > 0) {
#pragma unroll
    for (int u = 0; u < 3; ++u)
#pragma unroll
      for (int i = 0; i < IPS; ++i) issue1(min(u, nkt - 1), u, i);
  }
  // 256 register writes per wavefront, under the latency of the first loads.  (The empty statements keep them here and make the
  // values opaque: left to itself the compiler zeroed the registers ahead of the loads and a second time behind them, 1.3 us
  // of a 65 us product.)
  f32x16_t acc[TA][4];
#pragma unroll
  for (int i = 0; i < TA; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
      asm volatile("" : "+a"(acc[i][j]));
    }
  if (nkt > 0) {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * IPS) : "memory");
    asm volatile("s_barrier" ::: "memory");
#pragma unroll
    for (int q = 0; q < IPS; ++q) rd(F0, q, 0u, c0{});
  }
  auto mf = [&](const fset& X, int n) {
    const int i = n >> 2, j = (n & 3) ^ ((i & 1) ? 3 : 0);   // a block of B stays for two MFMAs in a row
    PQ_MFMA_BF16_ACC(acc[i][j], X.op(i), X.op(TA + j));
  };
  for (int kt = 0; kt < nkt; ++kt) {
    const uint32_t so = (uint32_t)(kt & 3) * STG, sn = (uint32_t)((kt + 1) & 3) * STG;
    const int ktl = min(kt + 3, nkt - 1), sl = (kt + 3) & 3;
    F0.wait_all();
#pragma unroll
    for (int n = 0; n < NM / 2; ++n) {                 // (with TA = 3 one block more than MFMAs to hide it behind)
      mf(F0, n);
      rd(F1, n, so, c1{});
      if (TA == 3 && n == 0) rd(F1, NM / 2, so, c1{});
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(IPS) : "memory");   // the wavefront's own loads of stage kt+1 have landed
    asm volatile("s_barrier" ::: "memory");            // everybody's have; nobody reads stage kt-1 any more
#pragma unroll
    for (int n = NM / 2; n < NM; ++n) {
      mf(F0, n);
      issue1(ktl, sl, n - NM / 2);
      if (TA == 3 && n == NM / 2) issue1(ktl, sl, NM / 2);
    }
    F1.wait_all();
#pragma unroll
    for (int n = 0; n < NM; ++n) {
      mf(F1, n);
      if (n < IPS) rd(F0, n, sn, c0{});                // past the last stage: a slot nobody uses
    }
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  PQ_MFMA_SETTLE_FIRST();
#pragma unroll
  for (int i = 0; i < TA; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) asm volatile("" : "+a"(acc[i][j]));
  asm volatile("s_barrier" ::: "memory");

  // ---- epilogue ----------------------------------------------------------------------------------
  epi_state st;
  epi_begin(epi, st);
  float* slab = splitk_part ? splitk_part + (size_t)split * M * N : nullptr;
  const bool plain = !slab && epi.out_kind == PQ_OUT_F32 && !epi.col_div && !epi.maskW && !epi.accumulate && !epi.dot_comp &&
                     !epi.sign_bytes && !TWO;                 // uniform
  unsigned tid_e = threadIdx.x;
  asm volatile("" : "+v"(tid_e));
  const int lane_e = tid_e & 63, wave_e = tid_e >> 6;
  const int wm_e = (wave_e >> 1) * 32 * TA, wn_e = (wave_e & 1) * 128;
  unsigned char* wreg = smem + wave_e * STG;
  const int mlim = (!slab && epi.m_limit > 0 && epi.m_limit < M) ? epi.m_limit : M;
  const int nlim = (!slab && epi.n_limit > 0 && epi.n_limit < N) ? epi.n_limit : N;
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const int nb = TA == 3 && pass == 1 ? 1 : 2;       // 32-row blocks of this pass
#pragma unroll
    for (int ii = 0; ii < nb; ++ii)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int i = 2 * pass + ii;
          // (copy the elements out first: a vector element is not a bit_cast-able lvalue)
          const float w0 = acc[i][j][4 * g], w1 = acc[i][j][4 * g + 1], w2 = acc[i][j][4 * g + 2], w3 = acc[i][j][4 * g + 3];
          const i32x4_t o = {(int)__float_as_uint(w0), (int)__float_as_uint(w1), (int)__float_as_uint(w2), (int)__float_as_uint(w3)};
          const int rl = ii * 32 + (lane_e & 31);
          const uint32_t adw = (uint32_t)(size_t)(wreg + rl * 512 + (((j * 8 + 2 * g + (lane_e >> 5)) ^ (rl & 31)) << 4));
          // (asm with two wait states behind it: see the staged epilogue of mfma_gemm_kernel)
          asm volatile("ds_write_b128 %0, %1\n\ts_nop 1" ::"v"(adw), "v"(o) : "memory");
        }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    if (slab || plain) {
      char* outp = slab ? (char*)slab : (char*)epi.C;
      const size_t ldo = (slab ? (size_t)N : (size_t)epi.ldc) * 4;
#pragma unroll 4
      for (int it = 0; it < 16 * nb; ++it) {
        const int rl = it * 2 + (lane_e >> 5), c = lane_e & 31;
        uint4 v = *reinterpret_cast<const uint4*>(wreg + rl * 512 + ((c ^ (rl & 31)) << 4));
        if (!slab) {
          v.x = __float_as_uint(__fmul_rn(st.sc0, __uint_as_float(v.x)));
          v.y = __float_as_uint(__fmul_rn(st.sc0, __uint_as_float(v.y)));
          v.z = __float_as_uint(__fmul_rn(st.sc0, __uint_as_float(v.z)));
          v.w = __float_as_uint(__fmul_rn(st.sc0, __uint_as_float(v.w)));
        }
        const int m = m0 + wm_e + pass * 64 + rl, n = n0 + wn_e + c * 4;
        if (m < mlim && n < nlim) *reinterpret_cast<uint4*>(outp + (size_t)m * ldo + (size_t)n * 4) = v;
      }
    } else {
#pragma unroll 2
      for (int it = 0; it < 8 * nb; ++it) {
        const int rl = it * 4 + (lane_e >> 4), c = (lane_e & 15) * 2;
        const uint4 r0 = *reinterpret_cast<const uint4*>(wreg + rl * 512 + ((c ^ (rl & 31)) << 4));
        const uint4 r1 = *reinterpret_cast<const uint4*>(wreg + rl * 512 + (((c + 1) ^ (rl & 31)) << 4));
        const int m = m0 + wm_e + pass * 64 + rl, n = n0 + wn_e + c * 4;
        if (m < M && n < N) epi_vec8<false, TWO>(epi, st, m, n, r0, r1);
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
  }
  if (!slab) epi_end<256>(epi, st, red, blockIdx.x);
#endif
}

template <bool RAGGED, bool DUAL, bool TWO>
__global__ __launch_bounds__(256) void gemm_tn_w4_kernel(int M, int N, int K, pq_operand A, pq_operand B, pq_epilogue epi, int nbn,
                                                          int total_tiles, int kchunk, float* splitk_part, pq_second_arg<DUAL> second) {
  gemm_tn_w4_body<4, RAGGED, DUAL, TWO>(M, N, K, A, B, epi, nbn, total_tiles, kchunk, splitk_part, second);
}
template <bool RAGGED, bool DUAL>
__global__ __launch_bounds__(256) void gemm_tn_192_kernel(int M, int N, int K, pq_operand A, pq_operand B, pq_epilogue epi, int nbn,
                                                           int total_tiles, int kchunk, float* splitk_part, pq_second_arg<DUAL> second) {
  gemm_tn_w4_body<3, RAGGED, DUAL, false>(M, N, K, A, B, epi, nbn, total_tiles, kchunk, splitk_part, second);
}

template <int BM, int BN, int WGM, int WGN, int KB, bool WHOLE, bool TAIL, bool INT8, int AK, int BKIND, int AK2 = -1, int BK2 = -1, bool DUAL = false>
int launch_mfma(const pq_gemm_plan& pl, int M, int N, int K, const pq_operand& A, const pq_operand& B,
                const pq_epilogue& epi, hipStream_t s, float* part, const pq_gemm_group& grp, const pq_phase2& ph2,
                const pq_gemm_second* second = nullptr) {
  // grouped rows: every group may end in a partial tile, so at most ceil(rows / BM) + n_groups row tiles exist
  const int nbm = grp.mode == 1 ? (grp.max_rows + BM - 1) / BM + grp.n_groups : (M + BM - 1) / BM;
  const int nbn = (N + BN - 1) / BN;
  const int tiles = nbm * nbn;
  dim3 grid(tiles, pl.splits, DUAL ? 2 : 1), block(WGM * WGN * 64);
  mfma_gemm_kernel<BM, BN, WGM, WGN, KB, WHOLE, TAIL, INT8, AK, BKIND, AK2, BK2, DUAL><<<grid, block, 0, s>>>(
      M, N, K, A, B, epi, nbn, tiles, pl.kchunk, pl.splits > 1 ? part : nullptr, grp, ph2, second_arg<DUAL>(second));
  PQ_CHECK_LAUNCH("mfma_gemm_kernel");
  return PQ_OK;
}

template <bool INT8, int AK, int BKIND, int AK2 = -1, int BK2 = -1>
int launch_mfma_cfg(const pq_gemm_plan& pl, int M, int N, int K, const pq_operand& A, const pq_operand& B,
                    const pq_epilogue& epi, hipStream_t s, float* part, const pq_gemm_group& grp, const pq_phase2& ph2,
                    const pq_gemm_second* second = nullptr) {
  if (pl.bn != 256) return pq_launch_tile(pl, M, N, K, A, B, epi, s, part, grp, ph2, second);
  // rows of 16-byte chunks on 16-byte boundaries, as every width and section of this library has them
  const long aes = AK == PQ_SRC_KC8 ? 1 : 2, bes = BKIND == PQ_SRC_KC8 ? 1 : 2;
  constexpr bool bits = BKIND == PQ_SRC_BITS8 || BKIND == PQ_SRC_BITS16;
  if ((A.ld * aes) % 16 || ((uintptr_t)A.p % 16) || (AK == PQ_SRC_KS16 && M % 8) || ((uintptr_t)B.p % 16) ||
      (bits ? B.ld % 4 != 0 || K % 32 != 0 : (B.ld * bes) % 16 != 0 || (BKIND == PQ_SRC_KS16 && N % 8)))
    return pq_set_error(PQ_ERR_SHAPE, "GEMM operands must have 16-byte aligned rows");
  // weight gradients: the four-wavefront kernel (no per-row divisor, no int32 output)
  if constexpr (AK == PQ_SRC_KS16 && BKIND == PQ_SRC_KS16 && AK2 < 0) {
    const int nbm = (M + pl.bm - 1) / pl.bm, nbn = (N + 255) / 256;
    const bool dual = grp.mode == 3, ragged = K % 32 != 0 || pl.kchunk % 32 != 0;
    dim3 grid(nbm * nbn, pl.splits, dual ? 2 : 1);
    if ((grp.mode && !dual) || epi.row_div || epi.out_kind == PQ_OUT_I32) return pq_set_error(PQ_ERR_BAD_ARG, "no 256x256 weight-gradient kernel for this epilogue");
    float* p = pl.splits > 1 ? part : nullptr;
#define PQ_W4(R, D, T) gemm_tn_w4_kernel<R, D, T><<<grid, 256, 0, s>>>(M, N, K, A, B, epi, nbn, nbm * nbn, pl.kchunk, p, second_arg<D>(second))
#define PQ_192(R, D) gemm_tn_192_kernel<R, D><<<grid, 256, 0, s>>>(M, N, K, A, B, epi, nbn, nbm * nbn, pl.kchunk, p, second_arg<D>(second))
    if (pl.bm == 192) {                              // (never with a second destination)
      if (dual) { if (ragged) PQ_192(true, true); else PQ_192(false, true); }
      else if (ragged) PQ_192(true, false);
      else PQ_192(false, false);
    } else if (dual) { if (ragged) PQ_W4(true, true, false); else PQ_W4(false, true, false); }
    else if (epi.m_split > 0) { if (ragged) PQ_W4(true, false, true); else PQ_W4(false, false, true); }
    else if (ragged) PQ_W4(true, false, false);
    else PQ_W4(false, false, false);
#undef PQ_W4
#undef PQ_192
    PQ_CHECK_LAUNCH("gemm_tn_w4_kernel");
    return PQ_OK;
  } else {
    // whole steps (packed rows of whole 16 bytes): no tail to look for; whole tiles too: no validity masks in the second contraction
    constexpr int EPB = INT8 ? 128 : 64;
    const bool steps = K % EPB == 0 && pl.kchunk % EPB == 0 && (!bits || B.ld % 16 == 0);
    if constexpr (bits) {
      if (grp.mode != 0 && grp.mode != 3) return pq_set_error(PQ_ERR_BAD_ARG, "no grouped kernel for packed signs");
      const bool whole = grp.mode == 0 && steps && M % 128 == 0 && N % 256 == 0;
      if constexpr (AK == PQ_SRC_KC8 && AK2 < 0)
        if (grp.mode == 3) {
          if (steps) return launch_mfma<128, 256, 1, 4, 128, false, false, INT8, AK, BKIND, AK2, BK2, true>(pl, M, N, K, A, B, epi, s, part, grp, ph2, second);
          return launch_mfma<128, 256, 1, 4, 128, false, true, INT8, AK, BKIND, AK2, BK2, true>(pl, M, N, K, A, B, epi, s, part, grp, ph2, second);
        }
      if (grp.mode == 3) return pq_set_error(PQ_ERR_BAD_ARG, "no paired 128x256 kernel for these operand kinds");
      if (whole) return launch_mfma<128, 256, 1, 4, 128, true, false, INT8, AK, BKIND, AK2, BK2>(pl, M, N, K, A, B, epi, s, part, grp, ph2);
      if (steps) return launch_mfma<128, 256, 1, 4, 128, false, false, INT8, AK, BKIND, AK2, BK2>(pl, M, N, K, A, B, epi, s, part, grp, ph2);
      return launch_mfma<128, 256, 1, 4, 128, false, true, INT8, AK, BKIND, AK2, BK2>(pl, M, N, K, A, B, epi, s, part, grp, ph2);
    } else {
      if (grp.mode == 3) return pq_set_error(PQ_ERR_BAD_ARG, "no paired 256x256 kernel for these operand kinds");
      if (steps) return launch_mfma<256, 256, 2, 4, 128, false, false, INT8, AK, BKIND, AK2, BK2>(pl, M, N, K, A, B, epi, s, part, grp, ph2);
      return launch_mfma<256, 256, 2, 4, 128, false, true, INT8, AK, BKIND, AK2, BK2>(pl, M, N, K, A, B, epi, s, part, grp, ph2);
    }
  }
}

}  // namespace

// ---------------------------------------------------------------------------------------------
// Rank-r products with a long row dimension: C[M][128] = scale * A[M][K] B^T, bf16, A with the contraction index
// contiguous.  B is [128][K] (H = X A^T of the high-precision branch, Sec. 3.2) or, contraction-strided, [K][128]
// (dH = alpha dY B of its backward), then with sum(comp * (A B^T)) as a side result (d alpha).
// ---------------------------------------------------------------------------------------------
// With 128 output columns the tile engine has one workgroup per CU and two loads in flight per thread, so it runs as
// a chain of memory latencies, and it needs a split contraction with slabs to occupy the chip at all.  Here a
// workgroup of four wavefronts owns 64 (or 32) rows and the whole contraction: the operand tiles of a 64-element step
// ([64][128 B] of A, chunks swizzled by row as in the tile engine, then 16 KB of B: [128][128 B] the same way, or
// [64][256 B] as it lies in memory for the transposing LDS reads) go straight into a ring of six LDS stages, five
// steps ahead of the MFMAs, so about 120 KB per CU are in flight and nothing is reduced afterwards; one barrier per step.
constexpr int SK_BN = 128;

// BM = 64: wavefront w computes rows 32 (w >> 1) and columns 64 (w & 1), six stages of 24 KB.  BM = 32: one row block,
// wavefront w computes columns 32 w, seven stages of 20 KB (twice the workgroups for the same rows: B is streamed by
// twice as many CUs, A by each of them half as long).
// I8: int8 operands (128 contraction elements per 128-byte step, exact int32 accumulation) and the de-quantising
// epilogue of the INT8 high-precision branch: value = ((scale / row_div[m]) * acc) / col_div[n], each step rounded to fp32.
template <bool BTR, int BM, bool I8>
__global__ __launch_bounds__(256) void skinny_gemm_kernel(const void* __restrict__ A, long lda,
                                                         const void* __restrict__ B, long ldb, int M, int K,
                                                         uint16_t* __restrict__ C, long ldc, float scale,
                                                         const uint16_t* __restrict__ comp, long ld_comp,
                                                         double* __restrict__ partials, const float* __restrict__ row_div,
                                                         const float* __restrict__ col_div) {
#if defined(__HIP_DEVICE_COMPILE__)
  static_assert(BM == 64 || BM == 32, "one or two 32-row blocks");
  static_assert(!(I8 && BTR), "int8 operands are contraction-contiguous");
  constexpr int ES = I8 ? 1 : 2;                      // bytes per operand element
  constexpr int NA = BM / 8;                          // 1 KB load blocks of A per stage; B has 16
  constexpr int LPW = (NA + 16) / 4;                  // load blocks per wavefront and stage
  constexpr int NST = BM == 64 ? 6 : 7;               // ring stages
  constexpr int STAGE = (NA + 16) * 1024;
  constexpr int NJ = BM == 64 ? 2 : 1;                // 32-column blocks per wavefront
  static_assert((NA + 16) % 4 == 0 && NST * STAGE <= 150 * 1024, "even split of the loads; the ring fits LDS");
  __shared__ __attribute__((aligned(16))) unsigned char smem[NST * STAGE];
  __shared__ double red[4];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = blockIdx.x * BM;
  const int wr0 = BM == 64 ? (wv >> 1) * 32 : 0;      // the wavefront's rows and columns inside the tile
  const int wc0 = BM == 64 ? (wv & 1) * 64 : wv * 32;
  const int nkt = (K * ES) >> 7;
  const uint32_t lds0 = (uint32_t)(size_t)smem;

  // direct loads: lane l of a load lands at byte 16 l of its 1 KB block.  A, and a contraction-contiguous B: a block is
  // 8 rows x 128 B and lane l fetches physical chunk l & 7 of row 8 b + (l >> 3).  Contraction-strided B: a block is
  // 4 contraction rows x 256 B and lane l fetches physical chunk l & 15 of row 4 b + (l >> 4).
  const char* src[LPW];
  size_t adv[LPW];                                    // source bytes per contraction step
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int b = wv * LPW + i;                       // 0..NA-1: A, then 16 blocks of B
    if (BTR && b >= NA) {
      const int t = (b - NA) * 4 + (lane >> 4), pc = lane & 15;
      const int c = pc ^ (4 * (t & 3));
      src[i] = (const char*)B + ((size_t)t * ldb + c * 8) * 2;
      adv[i] = (size_t)64 * ldb * 2;
    } else {
      const int r = (b < NA ? b : b - NA) * 8 + (lane >> 3), pc = lane & 7;
      const int c = pc ^ ((r ^ (r >> 3)) & 7);
      src[i] = b < NA ? (const char*)A + ((size_t)min(m0 + r, M - 1) * lda) * ES + c * 16   // rows past the end: the last row
                      : (const char*)B + ((size_t)r * ldb) * ES + c * 16;
      adv[i] = 128;
    }
  }
  auto issue = [&](int kt, int stage) {
#pragma unroll
    for (int i = 0; i < LPW; ++i)
      __builtin_amdgcn_global_load_lds(src[i] + (size_t)kt * adv[i], PQ_LDS_PTR(smem + stage * STAGE + (wv * LPW + i) * 1024), 16, 0, 0);
  };

  // fragment addresses in stage 0.  A (and a contraction-contiguous B): row l & 31 of the wavefront's block, logical
  // chunk 2 ks + (l >> 5).  Contraction-strided B: the transposing read takes, per lane, the address of four
  // consecutive columns in contraction row 8 (l >> 5) + ((l & 15) >> 2) (+ 4 for the second half of the operand).
  const int h = lane >> 5;
  uint32_t adA[4], adB[NJ][BTR ? 1 : 4];
  {
    const int ra = wr0 + (lane & 31);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) adA[ks] = lds0 + ra * 128 + ((((2 * ks + h) ^ ra ^ (ra >> 3)) & 7) << 4);
    if constexpr (BTR) {
      const int tl = 8 * h + ((lane & 15) >> 2), cl = 16 * ((lane >> 4) & 1) + 4 * (lane & 3), sw = 4 * ((lane & 15) >> 2);
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int col = wc0 + 32 * j + cl;
        adB[j][0] = lds0 + NA * 1024 + tl * 256 + (((col >> 3) ^ sw) << 4) + (col & 7) * 2;
      }
    } else {
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int rb = wc0 + j * 32 + (lane & 31);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) adB[j][ks] = lds0 + NA * 1024 + rb * 128 + ((((2 * ks + h) ^ rb ^ (rb >> 3)) & 7) << 4);
      }
    }
  }
  using acc_t = typename std::conditional<I8, i32x16_t, f32x16_t>::type;
  acc_t acc[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[j][v] = 0;

#pragma unroll
  for (int st = 0; st < NST - 1; ++st) issue(min(st, nkt - 1), st);   // steps past the end: the last one again, never read
  int st = 0;
  for (int kt = 0; kt < nkt; ++kt) {
    // all but the NST - 2 latest steps have landed: this step's tiles are there (for this wavefront; the barrier makes
    // it everybody's), and every wavefront is past its reads of the stage that is refilled next
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 2) * LPW) : "memory");
    asm volatile("s_barrier" ::: "memory");
    issue(min(kt + NST - 1, nkt - 1), st == 0 ? NST - 1 : st - 1);
    const uint32_t so = (uint32_t)(st * STAGE);
    i32x4_t fa[4];
    if constexpr (BTR) {
      constexpr int RPS = 1 + 2 * NJ;                 // LDS reads per sub-step
      pq_i32x2 hb[2][2 * NJ];                         // two sub-steps of B in flight: [parity][2 j + half]
      uint32_t pb[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) pb[j] = adB[j][0] + so;
#define PQ_SK_READ(ks)                                                                      \
  do {                                                                                      \
    PQ_DS_READ128(fa[ks], adA[ks] + so, 0);                                                 \
    PQ_DS_READ_TR(hb[(ks) & 1][0], pb[0], (ks) * 4096);                                      \
    PQ_DS_READ_TR(hb[(ks) & 1][1], pb[0], (ks) * 4096 + 1024);                               \
    if constexpr (NJ == 2) {                                                                \
      PQ_DS_READ_TR(hb[(ks) & 1][2 * (NJ - 1)], pb[NJ - 1], (ks) * 4096);                    \
      PQ_DS_READ_TR(hb[(ks) & 1][2 * (NJ - 1) + 1], pb[NJ - 1], (ks) * 4096 + 1024);         \
    }                                                                                       \
  } while (0)
#define PQ_SK_MFMA(ks, NOUT)                                                                                      \
  do {                                                                                                            \
    if constexpr (NJ == 2)                                                                                        \
      asm volatile("s_waitcnt lgkmcnt(%5)"                                                                        \
                   : "+v"(fa[ks]), "+v"(hb[(ks) & 1][0]), "+v"(hb[(ks) & 1][1]), "+v"(hb[(ks) & 1][2 * (NJ - 1)]),  \
                     "+v"(hb[(ks) & 1][2 * (NJ - 1) + 1])                                                         \
                   : "n"(NOUT));                                                                                  \
    else                                                                                                          \
      asm volatile("s_waitcnt lgkmcnt(%3)" : "+v"(fa[ks]), "+v"(hb[(ks) & 1][0]), "+v"(hb[(ks) & 1][1]) : "n"(NOUT)); \
    _Pragma("unroll") for (int j = 0; j < NJ; ++j) {                                                              \
      const i32x4_t b = {hb[(ks) & 1][2 * j][0], hb[(ks) & 1][2 * j][1], hb[(ks) & 1][2 * j + 1][0], hb[(ks) & 1][2 * j + 1][1]}; \
      PQ_MFMA_BF16(acc[j], fa[ks], b);                                                                            \
    }                                                                                                             \
  } while (0)
      PQ_SK_READ(0);
      PQ_SK_READ(1);
      PQ_SK_MFMA(0, RPS);
      PQ_SK_READ(2);
      PQ_SK_MFMA(1, RPS);
      PQ_SK_READ(3);
      PQ_SK_MFMA(2, RPS);
      PQ_SK_MFMA(3, 0);
#undef PQ_SK_READ
#undef PQ_SK_MFMA
    } else {
      constexpr int RPS = 1 + NJ;
      i32x4_t fb[NJ][4];
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        PQ_DS_READ128(fa[ks], adA[ks] + so, 0);
#pragma unroll
        for (int j = 0; j < NJ; ++j) PQ_DS_READ128(fb[j][ks], adB[j][ks] + so, 0);
      }
#define PQ_SK_MFMA(ks)                                                                                             \
  do {                                                                                                             \
    if constexpr (NJ == 2)                                                                                         \
      asm volatile("s_waitcnt lgkmcnt(%3)" : "+v"(fa[ks]), "+v"(fb[0][ks]), "+v"(fb[NJ - 1][ks]) : "n"((3 - (ks)) * RPS)); \
    else                                                                                                           \
      asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(fa[ks]), "+v"(fb[0][ks]) : "n"((3 - (ks)) * RPS));              \
    _Pragma("unroll") for (int j = 0; j < NJ; ++j) {                                                               \
      if constexpr (I8) PQ_MFMA_I8(acc[j], fa[ks], fb[j][ks]);                                                     \
      else PQ_MFMA_BF16(acc[j], fa[ks], fb[j][ks]);                                                                \
    }                                                                                                              \
  } while (0)
      PQ_SK_MFMA(0);
      PQ_SK_MFMA(1);
      PQ_SK_MFMA(2);
      PQ_SK_MFMA(3);
#undef PQ_SK_MFMA
    }
    st = st == NST - 1 ? 0 : st + 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the redundant loads of the last steps are done before the workgroup ends
  pq_mfma_settle(acc);

  // the B fragment was the first MFMA operand: lane l holds row l & 31, register v column 8 (v >> 2) + 4 (l >> 5) + (v & 3)
  const int m = m0 + wr0 + (lane & 31);
  double psum = 0.0;
  if (m < M) {
    const float sc = row_div ? scale / row_div[m] : scale;
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int n = wc0 + j * 32 + 8 * g + 4 * h;
        if constexpr (I8) {
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = __fmul_rn(sc, (float)acc[j][4 * g + e]);
          if (col_div) {                             // uniform
            const float4 cd = *reinterpret_cast<const float4*>(col_div + n);
            v[0] = v[0] / cd.x; v[1] = v[1] / cd.y; v[2] = v[2] / cd.z; v[3] = v[3] / cd.w;
          }
          *reinterpret_cast<uint2*>(C + (size_t)m * ldc + n) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
          continue;
        }
        if (comp) {                                  // uniform
          const uint2 u = *reinterpret_cast<const uint2*>(comp + (size_t)m * ld_comp + n);
          psum += (double)__uint_as_float(u.x << 16) * (double)acc[j][4 * g];
          psum += (double)__uint_as_float(u.x & 0xFFFF0000u) * (double)acc[j][4 * g + 1];
          psum += (double)__uint_as_float(u.y << 16) * (double)acc[j][4 * g + 2];
          psum += (double)__uint_as_float(u.y & 0xFFFF0000u) * (double)acc[j][4 * g + 3];
        }
        const float v0 = __fmul_rn(sc, (float)acc[j][4 * g]), v1 = __fmul_rn(sc, (float)acc[j][4 * g + 1]);
        const float v2 = __fmul_rn(sc, (float)acc[j][4 * g + 2]), v3 = __fmul_rn(sc, (float)acc[j][4 * g + 3]);
        *reinterpret_cast<uint2*>(C + (size_t)m * ldc + n) = make_uint2(pack_bf16x2(v0, v1), pack_bf16x2(v2, v3));
      }
  }
  if (partials) {                                    // uniform: one partial sum per workgroup, added in a fixed order
    const double t = block_sum_d<256>(psum, red);
    if (tid == 0) partials[blockIdx.x] = t;
  }
#endif
}

// The two weight gradients of the rank-128 branch, dB = alpha dY^T H and dA = dH^T X (Sec. 3.2, STE backward): the
// contraction runs over the tokens and both operands are stored token-major.  Same ring as above with both tiles as
// they lie in memory ([64 tokens][128 B] of the wide operand's 64 columns, [64 tokens][256 B] of the rank-128 one)
// and transposing LDS reads for both.  A workgroup owns 64 columns of the wide operand and one of 4 to 16 token
// ranges (blockIdx.y), and writes a 64 x 128 fp32 tile of that range's slab; blockIdx.z selects the problem.  For dA the wide
// operand is X, so the tile is the transpose of the output's and is stored transposed (dA is [128][d_in]).
struct skt_problem {
  const uint16_t* W;   // wide operand [T][ldw], M columns used
  long ldw;
  const uint16_t* R;   // rank-128 operand [T][ldr]
  long ldr;
  int M;               // multiple of 64
  int trans;           // 0: slab[split][M][128], 1: slab[split][128][M]
  float* slab;
};

__global__ __launch_bounds__(256) void skinny_tn_pair_kernel(skt_problem p0, skt_problem p1, int tokens_per_split) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int NST = 6, LPW = 6, STAGE = 24 * 1024;
  __shared__ __attribute__((aligned(16))) unsigned char smem[NST * STAGE];
  const skt_problem& p = blockIdx.z ? p1 : p0;        // uniform
  const int m0 = blockIdx.x * 64;
  if (m0 >= p.M) return;                              // uniform, ahead of every barrier
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int split = blockIdx.y;
  const size_t kb = (size_t)split * tokens_per_split;
  const int nkt = tokens_per_split >> 6;
  const uint32_t lds0 = (uint32_t)(size_t)smem;
  const int wr0 = (wv >> 1) * 32, wc0 = (wv & 1) * 64;

  // direct loads, lane l at byte 16 l of a 1 KB block.  Wide operand: a block is 8 tokens x 128 B, lane l fetches
  // physical chunk l & 7 of token 8 b + (l >> 3); rank-128 operand: 4 tokens x 256 B, chunk l & 15 of token 4 b + (l >> 4).
  // Chunks are XOR-swizzled by the token's two low bits so that the transposing reads spread over the banks.
  const char* src[LPW];
  size_t adv[LPW];
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int b = wv * LPW + i;                       // 0..7: wide operand, 8..23: rank-128 operand
    if (b < 8) {
      const int t = b * 8 + (lane >> 3), pc = lane & 7;
      const int c = pc ^ (2 * (t & 3));
      src[i] = (const char*)p.W + ((kb + t) * p.ldw + m0 + c * 8) * 2;
      adv[i] = (size_t)64 * p.ldw * 2;
    } else {
      const int t = (b - 8) * 4 + (lane >> 4), pc = lane & 15;
      const int c = pc ^ (4 * (t & 3));
      src[i] = (const char*)p.R + ((kb + t) * p.ldr + c * 8) * 2;
      adv[i] = (size_t)64 * p.ldr * 2;
    }
  }
  auto issue = [&](int kt, int stage) {
#pragma unroll
    for (int i = 0; i < LPW; ++i)
      __builtin_amdgcn_global_load_lds(src[i] + (size_t)kt * adv[i], PQ_LDS_PTR(smem + stage * STAGE + (wv * LPW + i) * 1024), 16, 0, 0);
  };

  // transposing reads: per lane the address of four consecutive columns in token 8 (l >> 5) + ((l & 15) >> 2) of a
  // 16-token sub-step (+ 4 tokens for the second half of the operand)
  const int h = lane >> 5, q = (lane & 15) >> 2;
  const int tl = 8 * h + q, cl = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  uint32_t adW, adR[2];
  {
    const int col = wr0 + cl;
    adW = lds0 + tl * 128 + ((((col >> 3) ^ (2 * q)) & 7) << 4) + (col & 7) * 2;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int cr = wc0 + 32 * j + cl;
      adR[j] = lds0 + 8 * 1024 + tl * 256 + (((cr >> 3) ^ (4 * q)) << 4) + (cr & 7) * 2;
    }
  }
  f32x16_t acc[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[j][v] = 0.0f;

#pragma unroll
  for (int st = 0; st < NST - 1; ++st) issue(min(st, nkt - 1), st);
  int st = 0;
  for (int kt = 0; kt < nkt; ++kt) {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 2) * LPW) : "memory");
    asm volatile("s_barrier" ::: "memory");
    issue(min(kt + NST - 1, nkt - 1), st == 0 ? NST - 1 : st - 1);
    const uint32_t so = (uint32_t)(st * STAGE);
    const uint32_t pw = adW + so, pr0 = adR[0] + so, pr1 = adR[1] + so;
    pq_i32x2 hw[2][2], hr[2][4];                      // two sub-steps in flight: [parity][...]
#define PQ_SKT_READ(ks)                                                     \
  do {                                                                      \
    PQ_DS_READ_TR(hw[(ks) & 1][0], pw, (ks) * 2048);                         \
    PQ_DS_READ_TR(hw[(ks) & 1][1], pw, (ks) * 2048 + 512);                   \
    PQ_DS_READ_TR(hr[(ks) & 1][0], pr0, (ks) * 4096);                        \
    PQ_DS_READ_TR(hr[(ks) & 1][1], pr0, (ks) * 4096 + 1024);                 \
    PQ_DS_READ_TR(hr[(ks) & 1][2], pr1, (ks) * 4096);                        \
    PQ_DS_READ_TR(hr[(ks) & 1][3], pr1, (ks) * 4096 + 1024);                 \
  } while (0)
#define PQ_SKT_MFMA(ks, NOUT)                                                                                    \
  do {                                                                                                           \
    asm volatile("s_waitcnt lgkmcnt(%6)"                                                                         \
                 : "+v"(hw[(ks) & 1][0]), "+v"(hw[(ks) & 1][1]), "+v"(hr[(ks) & 1][0]), "+v"(hr[(ks) & 1][1]),   \
                   "+v"(hr[(ks) & 1][2]), "+v"(hr[(ks) & 1][3])                                                  \
                 : "n"(NOUT));                                                                                   \
    const i32x4_t fw = {hw[(ks) & 1][0][0], hw[(ks) & 1][0][1], hw[(ks) & 1][1][0], hw[(ks) & 1][1][1]};         \
    const i32x4_t f0 = {hr[(ks) & 1][0][0], hr[(ks) & 1][0][1], hr[(ks) & 1][1][0], hr[(ks) & 1][1][1]};         \
    const i32x4_t f1 = {hr[(ks) & 1][2][0], hr[(ks) & 1][2][1], hr[(ks) & 1][3][0], hr[(ks) & 1][3][1]};         \
    PQ_MFMA_BF16(acc[0], fw, f0);                                                                                \
    PQ_MFMA_BF16(acc[1], fw, f1);                                                                                \
  } while (0)
    PQ_SKT_READ(0);
    PQ_SKT_READ(1);
    PQ_SKT_MFMA(0, 6);
    PQ_SKT_READ(2);
    PQ_SKT_MFMA(1, 6);
    PQ_SKT_READ(3);
    PQ_SKT_MFMA(2, 6);
    PQ_SKT_MFMA(3, 0);
#undef PQ_SKT_READ
#undef PQ_SKT_MFMA
    st = st == NST - 1 ? 0 : st + 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  pq_mfma_settle(acc);

  // lane l holds row l & 31 (a column of the wide operand), register v column 8 (v >> 2) + 4 (l >> 5) + (v & 3)
  const int m = m0 + wr0 + (lane & 31);
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int n = wc0 + j * 32 + 8 * g + 4 * h;
      if (p.trans) {                                  // uniform
#pragma unroll
        for (int e = 0; e < 4; ++e) p.slab[((size_t)split * SK_BN + n + e) * p.M + m] = acc[j][4 * g + e];
      } else {
        *reinterpret_cast<float4*>(p.slab + ((size_t)split * p.M + m) * SK_BN + n) =
            make_float4(acc[j][4 * g], acc[j][4 * g + 1], acc[j][4 * g + 2], acc[j][4 * g + 3]);
      }
    }
#endif
}

// Shapes, alignments and epilogues the kernel above takes: 128 columns, whole 64-element steps, a plain bf16 store,
// optionally with the dot product against a bf16 matrix of the output's shape.
bool pq_skinny_applies(int M, int N, int K, const pq_operand& A, const pq_operand& B, const pq_epilogue& e) {
  const bool btr = B.kind == PQ_SRC_KS16;
  const bool i8 = A.kind == PQ_SRC_KC8 && B.kind == PQ_SRC_KC8;
  const bool b16 = A.kind == PQ_SRC_KC16 && (B.kind == PQ_SRC_KC16 || btr);
  const long es = i8 ? 1 : 2;
  if (!(i8 || b16)) return false;
  if (!(M >= 1024 && N == SK_BN && K * es >= 128 && (K * es) % 128 == 0 && A.ld >= K && B.ld >= (btr ? N : K) &&
        (A.ld * es) % 16 == 0 && (B.ld * es) % 16 == 0 && ((uintptr_t)A.p % 16) == 0 && ((uintptr_t)B.p % 16) == 0))
    return false;
  if (!(e.out_kind == PQ_OUT_BF16 && e.ldc >= N && (e.ldc * 2) % 8 == 0 && ((uintptr_t)e.C % 8) == 0 && !e.sign_bytes && !e.maskW &&
        !e.accumulate && !e.dev_scale))
    return false;
  if (i8) return !e.dot_comp && !e.partials && (!e.col_div || ((uintptr_t)e.col_div % 16) == 0);   // de-quantising epilogue
  return !e.row_div && !e.col_div &&
         (!e.dot_comp || (e.comp_kind == PQ_OUT_BF16 && e.partials && e.ld_comp >= N && (e.ld_comp * 2) % 8 == 0 &&
                          ((uintptr_t)e.dot_comp % 8) == 0)) &&
         (e.dot_comp || !e.partials);
}

#ifndef PQ_SK_ROWS
#define PQ_SK_ROWS 32
#endif
int pq_skinny_blocks(int M) { return (M + PQ_SK_ROWS - 1) / PQ_SK_ROWS; }

int pq_launch_skinny(int M, int K, const pq_operand& A, const pq_operand& B, const pq_epilogue& e, hipStream_t s, int prof_label) {
  pq_prof_scope prof(prof_label, s);
  const dim3 grid(pq_skinny_blocks(M)), block(256);
  if (A.kind == PQ_SRC_KC8)
    skinny_gemm_kernel<false, PQ_SK_ROWS, true><<<grid, block, 0, s>>>(A.p, A.ld, B.p, B.ld, M, K, (uint16_t*)e.C, e.ldc, e.scale, nullptr, 0,
                                                                       nullptr, e.row_div, e.col_div);
  else if (B.kind == PQ_SRC_KS16)
    skinny_gemm_kernel<true, PQ_SK_ROWS, false><<<grid, block, 0, s>>>(A.p, A.ld, B.p, B.ld, M, K, (uint16_t*)e.C, e.ldc, e.scale,
                                                                       (const uint16_t*)e.dot_comp, e.ld_comp, e.partials, nullptr, nullptr);
  else
    skinny_gemm_kernel<false, PQ_SK_ROWS, false><<<grid, block, 0, s>>>(A.p, A.ld, B.p, B.ld, M, K, (uint16_t*)e.C, e.ldc, e.scale,
                                                                        (const uint16_t*)e.dot_comp, e.ld_comp, e.partials, nullptr, nullptr);
  PQ_CHECK_LAUNCH("skinny_gemm_kernel");
  return PQ_OK;
}

// Tile shape and contraction split for one GEMM: the smallest of the times (us) that the kernels were measured to take, c the
// workgroups a CU has to take one after the other:
//   64x64:   5 + 0.25 c per 128-byte step + 1 per further workgroup
//   128x128: 6 + 0.76 per step alone on a CU (int8 0.85), 0.58 c (0.61) when two workgroups share it, + 2.4 per further workgroup
//   256x256: c (9.5 + 1.38 per step); split only while the tiles are at most half of the CUs: beyond that more active CUs
//            lower the clock instead
//   192x256, weight gradients: c (9 + 1.19 per step): of use where 256x256 tiles leave a third of the CUs idle, or of the last
//            round (5504x2048 over 8192 tokens 216 -> 188, two such in one launch 383 -> 338; 5076x2048 over 2048 72 -> 65)
//   128x256, packed signs: 6 + 0.7 per step alone on a CU (int8 6.5 + 0.8; up to 0.12 more as the CUs fill up), u workgroups to a
//            CU 6 + 0.75 u per step (0.83 u) + 3 per workgroup behind the first.  These times count from 1024 columns or 192 tiles on,
//            512 rows and four steps; narrower and shorter outputs, where the two sizes of tiles measured 0.98-1.24 x
//            of each other either way, take it where 256x256 would have been the choice
//   a split: its slabs written at 10 TB/s (the caches take part of them), then 2 + slabs and result at 7 TB/s, at least 4
// Fitted to 997 timings of 141 shapes (64 to 16384 rows, 16 to 8192 columns, contractions of 16 to 8192; int8, bf16 and
// packed-sign operands): the tile and split these pick are 1 to 3 % slower than the fastest of all, averaged over the shapes;
// 128x256 to 347 timings of its own (1.4 %) and 60 of split ones (1.6 %, with 4 us more for the second launch).
// (2048 x 2048 outputs over 2048 / 8192 tokens: 64x64 37 / 126, 128x128 35 / 109, 256x256 in four splits 43 / 82 with the
// reduction; 765 x 672 over 672: 7, 13, 22.)
static double est_tile(int bm, long wgs, long steps, bool int8) {
  const double c = (double)((wgs + 255) / 256);
  if (bm == 64) return (int8 ? 5.3 : 5.0) + c * steps * 0.25 + (c - 1.0);
  if (bm == 128) return (int8 ? 6.3 : 6.0) + (wgs <= 256 ? steps * (int8 ? 0.85 : 0.76) : c * steps * (int8 ? 0.61 : 0.58)) + 2.4 * (c - 1.0);
  return c * (9.5 + steps * 1.38);
}
static double est_reduce(int splits, double elems) {
  if (splits <= 1) return 0.0;
  const double t = 2.0 + (4.0 * splits + 3.0) * elems / 7.0e6;
  return 4.0 * splits * elems / 1.0e7 + (t > 4.0 ? t : 4.0);
}

// Packed signs on 128x256 tiles: n tiles, two to a CU at a time.
static double est_signs(long n, long steps, bool int8) {
  const double u = (double)((n + 255) / 256);
  if (u == 1.0) return (int8 ? 6.5 + 0.8 * steps : 6.0 + 0.7 * steps) + (n > 128 ? 0.12 * (n - 128) / 128.0 * steps : 0.0);
  return 6.0 + u * steps * (int8 ? 0.83 : 0.75) + 3.0 * (u - 1.0);
}

// Weight gradients on 192x256 tiles, never split.
static double est_192(long tiles, long steps) {
  const double c = (double)((tiles + 255) / 256);
  return c * (9.0 + 1.19 * steps);
}

static pq_gemm_plan plan_search(int M, int N, int K, bool int8, bool may_split, pq_plan_kind kind) {
  const bool signs = kind == PQ_PLAN_SIGNS;
  pq_gemm_plan pl;
  memset(&pl, 0, sizeof(pl));
  pl.bm = pl.bn = 64;
  pl.splits = 1;
  pl.kchunk = K > 0 ? K : 1;
  const int epb = int8 ? 128 : 64;
  auto tiles_of = [&](int bm, int bn) { return (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
  const long t256 = tiles_of(256, 256);
  // 128x256 tiles of packed signs by their own times from 1024 columns or 192 tiles on (512 rows and four steps at least)
  const bool wide = M >= 512 && K > 3 * epb && (N >= 1024 || tiles_of(128, 256) >= 192);
  double best = 1e30;
  for (int c = 64; c <= 256; c *= 2) {
    if (c == 256 && !(M >= 256 && N >= 256)) continue;
    const int bm = (c == 256 && signs) ? 128 : c;
    const long tiles = tiles_of(bm, c);
    for (int want = 1; want <= 16; ++want) {
      if (want > 1 && (!may_split || K / want < 256 || tiles * want > 1024 || (c == 256 && (int8 || t256 > 128)))) break;
      const int chunk = want == 1 ? (K > 0 ? K : 1) : ((K + want - 1) / want + 255) / 256 * 256;   // whole 128-byte steps, at least two
      const int sp = want == 1 ? 1 : (K + chunk - 1) / chunk;
      const long steps = (chunk + epb - 1) / epb;
      const double t = (bm != c && wide ? est_signs(tiles * sp, steps, int8) + (sp > 1 ? 4.0 : 0.0) : est_tile(c, (c == 256 ? t256 : tiles) * sp, steps, int8)) +
                       est_reduce(sp, (double)M * N);
      if (t < best) { best = t; pl.bm = bm; pl.bn = c; pl.splits = sp; pl.kchunk = chunk; }
    }
  }
  if (kind == PQ_PLAN_WGRAD && M >= 192 && N >= 256) {
    const double t = est_192(tiles_of(192, 256), (K + 63) / 64);
    if (t < best) { best = t; pl.bm = 192; pl.bn = 256; pl.splits = 1; pl.kchunk = K > 0 ? K : 1; }
  }
  const long tiles = tiles_of(pl.bm, pl.bn);
  pl.red_blocks = pl.splits > 1 ? (int)(((size_t)M * (N / 8) + 255) / 256) : (int)tiles;
  pl.ws_bytes = pl.splits > 1 ? (size_t)pl.splits * M * N * sizeof(float) : 0;
  pl.us = best;
  return pl;
}
// The search is a pure function of its arguments and takes up to a microsecond; a call asks for a dozen plans (sizes of its
// sections, then the launches), most of them the ones it asked for before: the last answers are kept per thread.
static pq_gemm_plan pq_plan_gemm_impl(int M, int N, int K, bool int8, bool may_split, pq_plan_kind kind) {
  struct entry { int M, N, K, flags; pq_gemm_plan pl; };
  static thread_local entry cache[64];               // (zeroed: no plan has M = 0, see below)
  const int flags = (int8 ? 1 : 0) | (may_split ? 2 : 0) | (int)kind << 2;
  if (M <= 0) return plan_search(M, N, K, int8, may_split, kind);
  const uint32_t hsh = ((uint32_t)M * 2654435761u) ^ ((uint32_t)N * 2246822519u) ^ ((uint32_t)K * 3266489917u) ^ ((uint32_t)flags * 668265263u);
  entry& e = cache[(hsh ^ (hsh >> 15)) & 63u];
  if (e.M != M || e.N != N || e.K != K || e.flags != flags) e = entry{M, N, K, flags, plan_search(M, N, K, int8, may_split, kind)};
  return e.pl;
}
pq_gemm_plan pq_plan_gemm(int M, int N, int K, bool int8, bool split_int8, pq_plan_kind kind) {
  return pq_plan_gemm_impl(M, N, K, int8, !int8 || split_int8, kind);
}

static int check_scratch(size_t need, const pq_scratch& sk) {
  if (need == 0 || (sk.p && need <= sk.bytes)) return PQ_OK;
  return pq_set_error(PQ_ERR_WORKSPACE, "split contraction needs %zu bytes of scratch, its section has %zu", need, sk.p ? sk.bytes : 0);
}

// Two narrow products over the same contraction in one launch (dB and dA of the rank-r branch).  tn: rank 128 over many
// tokens, the streaming pair kernel (problem 1 runs transposed): four token ranges when that already gives a workgroup per
// CU (fewer slabs to write and add), up to sixteen for small matrices, never shorter than 256 tokens.  Otherwise 64x64 tiles,
// while they are not slower than a launch for each product with the tile it would choose: times as above, but no less than it
// takes to fetch the tiles' operands (20 TB/s out of the caches, 6.5 TB/s from 64 MB of operands on).  Over 286 shapes (300 to
// 16384 tokens, rank 16 to 1024) the choice costs 0.2 % of the whole step on average; 64x64 tiles always cost up to 26 % (16384
// tokens 4096 -> 1024, r = 512: 709 -> 846 us; this rule 690).
pq_pair_plan pq_plan_pair(int K, int M0, int N0, int M1, int N1) {
  pq_pair_plan p;
  memset(&p, 0, sizeof(p));
  int sp = 4;
  while (sp < 16 && (M0 / 64 + N1 / 64) * sp < 256 && K % (sp * 2 * 64) == 0 && K / (sp * 2) >= 256) sp *= 2;
  p.tn = N0 == SK_BN && M1 == SK_BN && M0 >= 64 && N1 >= 64 && M0 % 64 == 0 && N1 % 64 == 0 && K >= 2048 && K % (sp * 64) == 0;
  p.splits = sp;
  p.kchunk = K / sp;
  if (!p.tn) {
    const long tiles = (long)((M0 + 63) / 64) * ((N0 + 63) / 64) + (long)((M1 + 63) / 64) * ((N1 + 63) / 64);
    const double elems = (double)M0 * N0 + (double)M1 * N1;
    double best = 1e30;
    for (int want = 1; want <= 16; ++want) {
      if (want > 1 && (K / want < 256 || tiles * want > 1024)) break;
      const int chunk = want == 1 ? (K > 0 ? K : 1) : ((K + want - 1) / want + 255) / 256 * 256;
      const int n = want == 1 ? 1 : (K + chunk - 1) / chunk;
      const double t = est_tile(64, tiles * n, (chunk + 63) / 64, false) + est_reduce(n, elems);
      if (t < best) { best = t; p.splits = n; p.kchunk = chunk; }
    }
    const pq_gemm_plan p0 = pq_plan_gemm(M0, N0, K), p1 = pq_plan_gemm(M1, N1, K);
    const double rate = 2.0 * K * ((double)M0 + N0 + M1 + N1) > 64.0e6 ? 6.5e6 : 20.0e6;
    auto bound = [&](double us, long n, int bm, double reduce) {
      const double fetch = 5.0 + (double)n * ((K + 63) / 64) * bm * 256.0 / rate + reduce;
      return fetch > us ? fetch : us;
    };
    auto alone = [&](const pq_gemm_plan& q, int M, int N) {
      return bound(q.us, (long)((M + q.bm - 1) / q.bm) * ((N + q.bn - 1) / q.bn), q.bm, est_reduce(q.splits, (double)M * N));
    };
    if (alone(p0, M0, N0) + alone(p1, M1, N1) < bound(best, tiles, 64, est_reduce(p.splits, elems))) {
      p.apart = true;
      p.ws0 = p0.ws_bytes;
      p.ws1 = p1.ws_bytes;
      return p;
    }
  }
  p.ws0 = p.splits > 1 ? (size_t)p.splits * M0 * N0 * sizeof(float) : 0;
  p.ws1 = p.splits > 1 ? (size_t)p.splits * M1 * N1 * sizeof(float) : 0;
  return p;
}

static int check_epilogue(int M, const pq_operand& A, const pq_operand& B, const pq_epilogue& epi);
static pq_gemm_plan plan_call(int M, int N, int K, const pq_operand& A, const pq_operand& B, const pq_epilogue& epi, const pq_gemm_group& grp,
                              pq_scratch sk);
// A product on 64x64 tiles, not split: c is its launch.
static bool pq_plain_64(const pq_gemm_call& w, pq_scratch sk, pq_tile_call* c) {
  if (w.M <= 0 || w.N <= 0 || w.K <= 0 || check_epilogue(w.M, w.A, w.B, w.epi)) return false;
  *c = pq_tile_call{w.M, w.N, w.K, w.A, w.B, w.epi, {}, {}, nullptr};
  c->pl = plan_call(w.M, w.N, w.K, w.A, w.B, w.epi, c->grp, sk);
  return c->pl.bm == 64 && c->pl.bn == 64 && c->pl.splits == 1;
}
int pq_launch_gemm_pair_ks16(int K, int M0, int N0, const pq_operand& A0, const pq_operand& B0, float* C0, int ldc0, float scale0,
                             int M1, int N1, const pq_operand& A1, const pq_operand& B1, float* C1, int ldc1, float scale1,
                             hipStream_t s, int prof_label0, int prof_label1, pq_scratch sk0, pq_scratch sk1,
                             const pq_reduce_job* jobs, bool* jobs_done, const pq_grads* along) {
  if (jobs_done) *jobs_done = false;
  pq_epilogue e0;
  memset(&e0, 0, sizeof(e0));
  e0.C = C0; e0.ldc = ldc0; e0.out_kind = PQ_OUT_F32; e0.scale = scale0;
  pq_epilogue e1 = e0;
  e1.C = C1; e1.ldc = ldc1; e1.scale = scale1;
  const pq_pair_plan pp = pq_plan_pair(K, M0, N0, M1, N1);
  pq_reduce_job none;
  memset(&none, 0, sizeof(none));
  const int rb0 = (int)(((size_t)M0 * (N0 / 8) + 255) / 256), rb1 = (int)(((size_t)M1 * (N1 / 8) + 255) / 256);
  auto al = [](const pq_operand& o) { return o.kind == PQ_SRC_KS16 && (o.ld * 2) % 16 == 0 && ((uintptr_t)o.p % 16) == 0; };
  const bool one = M0 > 0 && N0 > 0 && M1 > 0 && N1 > 0 && K > 0 && al(A0) && al(B0) && al(A1) && al(B1) && A0.ld >= M0 && B0.ld >= N0 &&
                   A1.ld >= M1 && B1.ld >= N1 &&
                   (pp.splits == 1 || (sk0.p && sk1.p && ((uintptr_t)sk0.p % 16) == 0 && ((uintptr_t)sk1.p % 16) == 0));
  bool launched = false;
  if (along) {
    // (dW on 64x64 tiles, not split: those of dB and dA end with its own at the latest)
    pq_tile_call c[3], x;
    const pq_gemm_call &w = along->w, &xc = along->x;
    bool w_too = one && !pp.apart && !pp.tn && pq_plain_64(w, along->sk, &c[0]);
    if (w_too && pp.splits > 1) {
      // A split pair joins a dW of more than one workgroup per CU (1724 tokens 1984 -> 736, r = 32, INT8 branch: whole call 107.0 -> 101.0 us) or one
      // that it leaves at that; below, dW would lose its deep ring to it (3032 tokens 1504 -> 480, r = 16: 110.9 -> 114.4).
      auto tiles = [](int m, int n) { return (long)((m + 63) / 64) * ((n + 63) / 64); };
      const long nw = tiles(w.M, w.N);
      w_too = nw > 256 || nw + pp.splits * (tiles(M0, N0) + tiles(M1, N1)) <= 256;
    }
    const bool x_too = w_too && along->has_x && pq_plain_64(xc, along->sk, &x);
    if (along->has_x && !x_too)
      if (int rc = pq_launch_gemm(xc.M, xc.N, xc.K, xc.A, xc.B, xc.epi, s, xc.prof_label, along->sk, nullptr, &along->p2)) return rc;
    if (w_too) {
      if (int rc = check_scratch(pp.ws0, sk0)) return rc;
      if (int rc = check_scratch(pp.ws1, sk1)) return rc;
      pq_gemm_plan pl = c[0].pl;
      pl.splits = pp.splits; pl.kchunk = pp.kchunk;
      c[1] = pq_tile_call{M0, N0, K, A0, B0, e0, c[0].grp, pl, (float*)sk0.p};
      c[2] = pq_tile_call{M1, N1, K, A1, B1, e1, c[0].grp, pl, (float*)sk1.p};
      pq_prof_scope prof(w.prof_label, s);
      if (int rc = pq_launch_tile_grads(c, x_too ? &x : nullptr, x_too ? &along->p2 : nullptr, s)) return rc;
      launched = true;
    } else if (int rc = pq_launch_gemm(w.M, w.N, w.K, w.A, w.B, w.epi, s, w.prof_label, along->sk)) return rc;
  }
  if (!one || pp.apart) {
    if (int rc = pq_launch_gemm(M0, N0, K, A0, B0, e0, s, prof_label0, sk0)) return rc;
    return pq_launch_gemm(M1, N1, K, A1, B1, e1, s, prof_label1, sk1);
  }
  if (int rc = check_scratch(pp.ws0, sk0)) return rc;
  if (int rc = check_scratch(pp.ws1, sk1)) return rc;
  if (!launched) {
    pq_prof_scope prof(prof_label0, s);
    if (pp.tn) {
      skt_problem q0{(const uint16_t*)A0.p, A0.ld, (const uint16_t*)B0.p, B0.ld, M0, 0, (float*)sk0.p};
      skt_problem q1{(const uint16_t*)B1.p, B1.ld, (const uint16_t*)A1.p, A1.ld, N1, 1, (float*)sk1.p};
      const dim3 grid((M0 > N1 ? M0 : N1) / 64, pp.splits, 2);
      skinny_tn_pair_kernel<<<grid, 256, 0, s>>>(q0, q1, K / pp.splits);
      PQ_CHECK_LAUNCH("skinny_tn_pair_kernel");
    } else {
      pq_gemm_plan pl;
      memset(&pl, 0, sizeof(pl));
      pl.bm = pl.bn = 64; pl.splits = pp.splits; pl.kchunk = pp.kchunk;
      pq_gemm_group grp;
      memset(&grp, 0, sizeof(grp));
      grp.mode = 3;
      pq_gemm_second second{A1, B1, C1, ldc1, scale1, pp.splits > 1 ? (float*)sk1.p : nullptr, nullptr, M1, N1, (N1 + 63) / 64};
      pq_phase2 ph2;
      memset(&ph2, 0, sizeof(ph2));
      if (int rc = pq_launch_tile(pl, M0, N0, K, A0, B0, e0, s, (float*)sk0.p, grp, ph2, &second)) return rc;
    }
  }
  if (pp.splits > 1) {
    pq_prof_scope prof(PQP_SPLITK_REDUCE, s);
    splitk_reduce_pair_kernel<false><<<rb0 + rb1 + (jobs ? 2 : 0), 256, 0, s>>>(pp.splits, rb0, rb1, M0, N0, (const float*)sk0.p, e0, M1, N1,
                                                                        (const float*)sk1.p, e1, jobs ? jobs[0] : none,
                                                                        jobs ? jobs[1] : none);
    PQ_CHECK_LAUNCH("splitk_reduce_pair_kernel");
    if (jobs && jobs_done) *jobs_done = true;
  }
  return PQ_OK;
}

// Two products of the same sizes, kinds and epilogue but for C and the device scale (U and G of the FFN; dW_up and dW_gate) in
// one launch: one start and one tail instead of two, and together they fill the chip where each alone does not.
// (int8: U and G, with packed signs; otherwise dW_up and dW_gate)
pq_gemm_plan pq_plan_dual(int M, int N, int K, bool int8) { return pq_plan_gemm_impl(2 * M, N, K, int8, true, int8 ? PQ_PLAN_SIGNS : PQ_PLAN_WGRAD); }
int pq_launch_gemm_dual(int M, int N, int K, const pq_operand& A0, const pq_operand& B0, const pq_epilogue& e0, const pq_operand& A1,
                        const pq_operand& B1, void* C1, const float* dev_scale1, hipStream_t s, int prof_label, pq_scratch sk) {
  if (M <= 0 || N <= 0) return PQ_OK;
  const bool int8 = A0.kind == PQ_SRC_KC8;
  const pq_gemm_plan pl = pq_plan_dual(M, N, K, int8);
  if (int rc = check_scratch(pl.ws_bytes, sk)) return rc;
  if (e0.partials || e0.accumulate || e0.dot_comp || e0.sign_bytes || e0.maskW || e0.m_split || e0.n_limit % 4)
    return pq_set_error(PQ_ERR_BAD_ARG, "paired products take plain epilogues");
  float* part = (float*)sk.p;
  pq_gemm_group grp;
  memset(&grp, 0, sizeof(grp));
  grp.mode = 3;
  const pq_gemm_second second{A1, B1, C1, (int)e0.ldc, e0.scale, pl.splits > 1 ? part + (size_t)pl.splits * M * N : nullptr, dev_scale1,
                              M, N, (N + pl.bn - 1) / pl.bn};
  pq_phase2 ph2;
  memset(&ph2, 0, sizeof(ph2));
  {
    pq_prof_scope prof(prof_label, s);
    int rc;
    if (int8 && B0.kind == PQ_SRC_BITS8) rc = launch_mfma_cfg<true, PQ_SRC_KC8, PQ_SRC_BITS8>(pl, M, N, K, A0, B0, e0, s, part, grp, ph2, &second);
    else if (A0.kind == PQ_SRC_KS16 && B0.kind == PQ_SRC_KS16) rc = launch_mfma_cfg<false, PQ_SRC_KS16, PQ_SRC_KS16>(pl, M, N, K, A0, B0, e0, s, part, grp, ph2, &second);
    else return pq_set_error(PQ_ERR_BAD_ARG, "no paired kernel for operand kinds (%d, %d)", A0.kind, B0.kind);
    if (rc) return rc;
  }
  if (pl.splits > 1) {
    pq_prof_scope prof(PQP_SPLITK_REDUCE, s);
    pq_epilogue e1 = e0;
    e1.C = C1; e1.dev_scale = dev_scale1;
    pq_reduce_job none;
    memset(&none, 0, sizeof(none));
    const int rb = (int)(((size_t)M * (N / 8) + 255) / 256);
    if (int8) splitk_reduce_pair_kernel<true><<<2 * rb, 256, 0, s>>>(pl.splits, rb, rb, M, N, part, e0, M, N, second.part, e1, none, none);
    else splitk_reduce_pair_kernel<false><<<2 * rb, 256, 0, s>>>(pl.splits, rb, rb, M, N, part, e0, M, N, second.part, e1, none, none);
    PQ_CHECK_LAUNCH("splitk_reduce_pair_kernel");
  }
  return PQ_OK;
}

// Grouped contraction ranges (per-expert weight gradients): tile and pieces of every group's range (up to 8, of about 256
// indices or more, whose slabs a second launch adds), by the times above for segments of equal length.
struct mode2_plan { int bm, splits; };
static mode2_plan plan_mode2(int M, int N, int n_groups, int total_k) {
  mode2_plan p{64, 1};
  if (M <= 0 || N <= 0 || n_groups <= 0) return p;
  const long len = (total_k + n_groups - 1) / n_groups;
  double best = 1e30;
  for (int bm = 64; bm <= 128; bm *= 2) {
    const long tiles = (long)((M + bm - 1) / bm) * ((N + bm - 1) / bm) * n_groups;
    for (int sp = 1; sp <= 8; ++sp) {
      if (sp > 1 && (len / sp < 256 || tiles * sp > 1024)) break;
      const double t = est_tile(bm, tiles * sp, (len / sp + 63) / 64, false) + est_reduce(sp, (double)n_groups * M * N);
      if (t < best) { best = t; p.bm = bm; p.splits = sp; }
    }
  }
  return p;
}
size_t pq_mode2_ws_bytes(int M, int N, int n_groups, int total_k) {
  const int sp = plan_mode2(M, N, n_groups, total_k).splits;
  return sp > 1 ? (size_t)sp * n_groups * M * N * sizeof(float) : 0;
}

// what an epilogue asks for that no kernel does
static int check_epilogue(int M, const pq_operand& A, const pq_operand& B, const pq_epilogue& epi) {
  if ((epi.n_limit > 0 || epi.m_limit > 0) && (epi.accumulate || epi.maskW || epi.dot_comp || epi.n_limit % 4 != 0))
    return pq_set_error(PQ_ERR_BAD_ARG, "store limits go with plain stores and a column limit that is a multiple of 4");
  if (epi.m_split > 0 && (A.kind != PQ_SRC_KS16 || B.kind != PQ_SRC_KS16 || epi.out_kind != PQ_OUT_F32 || epi.accumulate || epi.maskW || epi.dot_comp ||
                          epi.m_limit || epi.n_limit || M % (2 * epi.m_split) != 0))
    return pq_set_error(PQ_ERR_BAD_ARG, "a second destination goes with plain fp32 weight gradients");
  if (epi.C2 && epi.m_split == 0 && (A.kind != PQ_SRC_KC8 || B.kind != PQ_SRC_KC8 || epi.out_kind != PQ_OUT_BF16 || !epi.accumulate || epi.split_int8 ||
                                     epi.m_limit || epi.n_limit))
    return pq_set_error(PQ_ERR_BAD_ARG, "a copy of the value goes with int8 products that accumulate");
  return PQ_OK;
}

// Tile, contraction split and scratch of a product; grp: plain (mode 0), row groups or contraction ranges.
static pq_gemm_plan plan_call(int M, int N, int K, const pq_operand& A, const pq_operand& B, const pq_epilogue& epi, const pq_gemm_group& grp,
                              pq_scratch sk) {
  const int ak = A.kind, bk = B.kind;
  const bool int8 = (ak == PQ_SRC_KC8);
  pq_gemm_plan pl = pq_plan_gemm(M, N, K, int8, epi.split_int8 != 0,
                                 bk == PQ_SRC_BITS8 || bk == PQ_SRC_BITS16                             ? PQ_PLAN_SIGNS
                                 : ak == PQ_SRC_KS16 && bk == PQ_SRC_KS16 && epi.m_split == 0 ? PQ_PLAN_WGRAD
                                                                                              : PQ_PLAN_ANY);
  if (grp.mode) {
    pl.splits = 1;
    pl.kchunk = K > 0 ? K : 1;
    pl.ws_bytes = 0;
    pl.bm = pl.bn = 64;
    // contraction ranges: pieces only for a plain fp32 output whose groups lie one behind the other
    if (grp.mode == 2) {
      const mode2_plan p2 = plan_mode2(M, N, grp.n_groups, K);
      pl.bm = pl.bn = p2.bm;
      if (p2.splits > 1 && sk.p && epi.out_kind == PQ_OUT_F32 && epi.ldc == N && grp.c_stride == (long)(epi.m_split ? epi.m_split : M) * N && N % 8 == 0 &&
          !epi.partials && !epi.dot_comp && !epi.sign_bytes && !epi.maskW && !epi.accumulate && !epi.row_div && !epi.col_div &&
          epi.m_limit == 0 && epi.n_limit == 0) {
        pl.splits = p2.splits;
        pl.red_blocks = (int)(((size_t)grp.n_groups * M * (N / 8) + 255) / 256);
        pl.ws_bytes = pq_mode2_ws_bytes(M, N, grp.n_groups, K);
      }
    }
    // row groups (expert segments): the tile by the same times, the
    // contraction of a product with few tiles split as for plain GEMMs.  A per-group column divisor is applied in the
    // GEMM's own epilogue only, so such products are not split.
    if (grp.mode == 1) {
      const bool narrow = N <= 128, wide = N >= 256 && K % 512 == 0 && epi.out_kind == PQ_OUT_BF16 && !epi.accumulate && !epi.row_div;
      // (N <= K: callers size the scratch for eight slabs as wide as the hidden states)
      const bool may = (narrow || wide) && N <= K && K >= 1024 && sk.p && !(epi.col_div && grp.coldiv_stride);
      const int epb = int8 ? 128 : 64;
      double best = 1e30;
      for (int bm = 64; bm <= 256; bm *= 2) {
        if (bm == 256 && !(N >= 256 && grp.max_rows >= 256)) continue;
        const long tiles = ((long)(grp.max_rows + bm - 1) / bm + (grp.n_groups + 1) / 2) * ((N + bm - 1) / bm);
        for (int want = 1; want <= 8; ++want) {
          if (want > 1 && (!may || tiles * want > 1024 || (bm == 256 && tiles > 128))) break;
          const int chunk = want == 1 ? K : ((K + want - 1) / want + 255) / 256 * 256;
          const int sp = (K + chunk - 1) / chunk;
          const double t = est_tile(bm, tiles * sp, (chunk + epb - 1) / epb, int8) + est_reduce(sp, (double)grp.max_rows * N);
          if (t < best) { best = t; pl.bm = pl.bn = bm; pl.splits = sp; pl.kchunk = chunk; }
        }
      }
      if (pl.splits > 1) {
        pl.red_blocks = (int)(((size_t)M * (N / 8) + 255) / 256);
        pl.ws_bytes = (size_t)pl.splits * M * N * sizeof(float);
      }
    }
  }
  return pl;
}

// The sum of a split contraction's slabs.  raw_int: the slabs are int32 accumulators.
static int reduce_call(int M, int N, const pq_epilogue& epi, const pq_gemm_group& grp, const pq_gemm_plan& pl, const float* part, bool raw_int,
                       hipStream_t s) {
  if (pl.splits > 1 && !epi.defer_reduce) {
    pq_prof_scope prof(PQP_SPLITK_REDUCE, s);
    const int Mred = grp.mode == 2 ? grp.n_groups * M : M;   // grouped ranges: the groups' outputs as one matrix
    if (raw_int) splitk_reduce_kernel<true, false><<<pl.red_blocks, 256, 0, s>>>(Mred, N, pl.splits, part, epi);
    else if (epi.m_split > 0) splitk_reduce_kernel<false, true><<<pl.red_blocks, 256, 0, s>>>(Mred, N, pl.splits, part, epi);
    else splitk_reduce_kernel<false, false><<<pl.red_blocks, 256, 0, s>>>(Mred, N, pl.splits, part, epi);
    PQ_CHECK_LAUNCH("splitk_reduce_kernel");
  }
  return PQ_OK;
}

int pq_launch_gemm(int M, int N, int K, const pq_operand& A, const pq_operand& B,
                   const pq_epilogue& epi, hipStream_t s, int prof_label, pq_scratch sk,
                   const pq_gemm_group* group, const pq_phase2* phase2) {
  if (M <= 0 || N <= 0) return PQ_OK;
  pq_gemm_group grp;
  memset(&grp, 0, sizeof(grp));
  if (group) grp = *group;
  pq_phase2 ph2;
  memset(&ph2, 0, sizeof(ph2));
  if (phase2) ph2 = *phase2;
  if (ph2.K2 > 0 && grp.mode) return pq_set_error(PQ_ERR_BAD_ARG, "a fused second contraction needs the plain MFMA engine");
  if (int rc = check_epilogue(M, A, B, epi)) return rc;
  // plain rank-128 products over many rows: the streaming kernel (callers that want per-block partial sums or the
  // slabs of a split contraction choose it themselves, since it changes how many of those there are)
  if (!grp.mode && ph2.K2 == 0 && !epi.partials && !epi.defer_reduce && pq_skinny_applies(M, N, K, A, B, epi))
    return pq_launch_skinny(M, K, A, B, epi, s, prof_label);
  const int ak = A.kind, bk = B.kind;
  const bool int8 = (ak == PQ_SRC_KC8);
  const pq_gemm_plan pl = plan_call(M, N, K, A, B, epi, grp, sk);
  if (int rc = check_scratch(pl.ws_bytes, sk)) return rc;
  float* part = (float*)sk.p;
  int rc;
  {
    pq_prof_scope prof(prof_label, s);   // the MFMA kernel alone; a split's reduction is timed under its own label
    if (ph2.K2 > 0) {
      if (!pq_plan_fuses(pl)) return pq_set_error(PQ_ERR_BAD_ARG, "a fused second contraction cannot be combined with a split contraction of 128x256 tiles");
      if (ak == PQ_SRC_KC8 && bk == PQ_SRC_BITS8 && ph2.A2.kind == PQ_SRC_KC16 && ph2.B2.kind == PQ_SRC_KC16)
        rc = launch_mfma_cfg<true, PQ_SRC_KC8, PQ_SRC_BITS8, PQ_SRC_KC16, PQ_SRC_KC16>(pl, M, N, K, A, B, epi, s, part, grp, ph2);
      else if (ak == PQ_SRC_KC16 && bk == PQ_SRC_BITS16 && ph2.A2.kind == PQ_SRC_KC16 && ph2.B2.kind == PQ_SRC_KS16)
        rc = launch_mfma_cfg<false, PQ_SRC_KC16, PQ_SRC_BITS16, PQ_SRC_KC16, PQ_SRC_KS16>(pl, M, N, K, A, B, epi, s, part, grp, ph2);
      else return pq_set_error(PQ_ERR_BAD_ARG, "no fused MFMA kernel for these operand kinds");
    } else if (ak == PQ_SRC_KC8 && bk == PQ_SRC_BITS8) rc = launch_mfma_cfg<true, PQ_SRC_KC8, PQ_SRC_BITS8>(pl, M, N, K, A, B, epi, s, part, grp, ph2);
    else if (ak == PQ_SRC_KC8 && bk == PQ_SRC_KC8) rc = launch_mfma_cfg<true, PQ_SRC_KC8, PQ_SRC_KC8>(pl, M, N, K, A, B, epi, s, part, grp, ph2);
    else if (ak == PQ_SRC_KC16 && bk == PQ_SRC_KC16) rc = launch_mfma_cfg<false, PQ_SRC_KC16, PQ_SRC_KC16>(pl, M, N, K, A, B, epi, s, part, grp, ph2);
    else if (ak == PQ_SRC_KC16 && bk == PQ_SRC_KS16) rc = launch_mfma_cfg<false, PQ_SRC_KC16, PQ_SRC_KS16>(pl, M, N, K, A, B, epi, s, part, grp, ph2);
    else if (ak == PQ_SRC_KC16 && bk == PQ_SRC_BITS16) rc = launch_mfma_cfg<false, PQ_SRC_KC16, PQ_SRC_BITS16>(pl, M, N, K, A, B, epi, s, part, grp, ph2);
    else if (ak == PQ_SRC_KS16 && bk == PQ_SRC_KS16) rc = launch_mfma_cfg<false, PQ_SRC_KS16, PQ_SRC_KS16>(pl, M, N, K, A, B, epi, s, part, grp, ph2);
    else return pq_set_error(PQ_ERR_BAD_ARG, "no MFMA kernel for operand kinds (%d, %d)", ak, bk);
  }
  if (rc != PQ_OK) return rc;
  // (with a second contraction the slabs are already floating-point numbers)
  return reduce_call(M, N, epi, grp, pl, part, int8 && ph2.K2 == 0, s);
}

// One 128x256 tile to a product of packed signs and nothing split: the output passes through the staged epilogue.
bool pq_gemm_swiglu_applies(int M, int N, int K) {
  if (M <= 0) return false;
  const pq_gemm_plan pl = pq_plan_gemm(M, N, K, false, false, PQ_PLAN_SIGNS);
  return pl.bm == 128 && pl.bn == 256 && pl.splits == 1;
}
int pq_launch_gemm_swiglu(int M, int N, int K, const pq_operand& A, const pq_operand& B, float scale, const float* dev_scale, const pq_gemm_act& act,
                          hipStream_t s, int prof_label) {
  if (!pq_gemm_swiglu_applies(M, N, K) || A.kind != PQ_SRC_KC16 || B.kind != PQ_SRC_BITS16 || N % 8 != 0 || K % 32 != 0 || B.ld % 4 != 0 || A.ld % 8 != 0 ||
      (uintptr_t)A.p % 16 || (uintptr_t)B.p % 16)
    return pq_set_error(PQ_ERR_BAD_ARG, "no product with the gated unit's derivative for M=%d N=%d K=%d", M, N, K);
  pq_epilogue e;
  memset(&e, 0, sizeof(e));
  e.ldc = N; e.out_kind = PQ_OUT_BF16; e.scale = scale; e.dev_scale = dev_scale;
  pq_gemm_group grp;
  memset(&grp, 0, sizeof(grp));
  pq_phase2 ph2;
  memset(&ph2, 0, sizeof(ph2));
  pq_prof_scope prof(prof_label, s);
  const int nbn = (N + 255) / 256, tiles = (M + 127) / 128 * nbn;
  if (K % 64 == 0 && B.ld % 16 == 0)
    mfma_gemm_kernel<128, 256, 1, 4, 128, false, false, false, PQ_SRC_KC16, PQ_SRC_BITS16, -1, -1, false, true>
        <<<tiles, 256, 0, s>>>(M, N, K, A, B, e, nbn, tiles, K, nullptr, grp, ph2, act);
  else
    mfma_gemm_kernel<128, 256, 1, 4, 128, false, true, false, PQ_SRC_KC16, PQ_SRC_BITS16, -1, -1, false, true>
        <<<tiles, 256, 0, s>>>(M, N, K, A, B, e, nbn, tiles, K, nullptr, grp, ph2, act);
  PQ_CHECK_LAUNCH("mfma_gemm_kernel");
  return PQ_OK;
}

// their launches (t, slabs side by side) and whether those can be one
static int plan_set(const pq_gemm_call* c, int n, pq_scratch sk, bool has_x, pq_tile_call* t, bool* together) {
  *together = false;
  if (n < 2 || n > 4 + has_x) return PQ_OK;
  size_t used = 0;
  for (int i = 0; i < n; ++i) {
    if (c[i].M <= 0 || c[i].N <= 0) return PQ_OK;
    if (int rc = check_epilogue(c[i].M, c[i].A, c[i].B, c[i].epi)) return rc;
    if (!c[i].grp && !c[i].epi.partials && pq_skinny_applies(c[i].M, c[i].N, c[i].K, c[i].A, c[i].B, c[i].epi)) return PQ_OK;   // (see pq_launch_gemm)
    t[i] = pq_tile_call{c[i].M, c[i].N, c[i].K, c[i].A, c[i].B, c[i].epi, {}, {}, nullptr};
    if (c[i].grp) t[i].grp = *c[i].grp;
    t[i].pl = plan_call(c[i].M, c[i].N, c[i].K, c[i].A, c[i].B, c[i].epi, t[i].grp, sk);
    if (t[i].pl.splits > 1) {
      t[i].part = (float*)((char*)sk.p + used);
      used += pq_align_up(t[i].pl.ws_bytes, 256);
    }
  }
  *together = used <= sk.bytes && pq_tile_set_applies(t, n - has_x, has_x ? &t[n - 1] : nullptr);
  return PQ_OK;
}
bool pq_gemm_set_shares(const pq_gemm_call* c, int n, pq_scratch sk, bool has_x) {
  pq_tile_call t[5];
  bool together;
  return plan_set(c, n, sk, has_x, t, &together) == PQ_OK && together;
}

int pq_launch_gemm_set(const pq_gemm_call* c, int n, hipStream_t s, pq_scratch sk, bool has_x) {
  pq_tile_call t[5];
  bool together;
  if (int rc = plan_set(c, n, sk, has_x, t, &together)) return rc;
  if (!together) {
    for (int i = 0; i < n; ++i)
      if (int rc = pq_launch_gemm(c[i].M, c[i].N, c[i].K, c[i].A, c[i].B, c[i].epi, s, c[i].prof_label, sk, c[i].grp)) return rc;
    return PQ_OK;
  }
  {
    pq_prof_scope prof(c[0].prof_label, s);
    if (int rc = pq_launch_tile_set(t, n - has_x, has_x ? &t[n - 1] : nullptr, s)) return rc;
  }
  for (int i = 0; i < n; ++i)
    if (int rc = reduce_call(t[i].M, t[i].N, t[i].epi, t[i].grp, t[i].pl, t[i].part, false, s)) return rc;
  return PQ_OK;
}

