// Internal launch interface between the C-ABI layer (pq_api.hip) and the kernel files.
#pragma once
#include "pq_common.h"

// ---- profiling labels (pq_api.hip) ---------------------------------------------------------
enum pq_prof_id {
  PQP_QUANT = 0, PQP_WSTATS, PQP_PACK, PQP_ROUTER, PQP_REDUCE,
  PQP_GEMM_ONEBIT, PQP_GEMM_HP_H, PQP_GEMM_HP_Y, PQP_GEMM_DH, PQP_GEMM_DX, PQP_GEMM_DX_HP,
  PQP_GEMM_DW, PQP_GEMM_DB, PQP_GEMM_DA, PQP_GEMM_OTHER, PQP_DECODE_PREP, PQP_DECODE_H, PQP_DECODE_MAIN, PQP_MOE_ROUTE, PQP_MOE_ELEMENTWISE, PQP_SWIGLU, PQP_GEMM_EXPERT, PQP_GLUE, PQP_SPLITK_REDUCE, PQP_NORM_QUANT, PQP_NORM_BWD, PQP_COUNT
};
struct pq_prof_scope {   // records an event pair around the launches made while it is alive
  int label; hipStream_t s; void* slot;
  pq_prof_scope(int label, hipStream_t s);
  ~pq_prof_scope();
};

// ---- pq_quant.hip -------------------------------------------------------------------------
// Per-token AbsMax INT8 quantiser.  Xt (optional, bf16) receives q/gamma, the de-quantised
// activation that the STE backward multiplies with.
int pq_launch_quant_act(const void* X, int dtype, int T, int K, int8_t* Xq, float* gamma,
                        uint16_t* Xt, hipStream_t s);
// RMSNorm fused with the quantiser: Xn (optional, I/O type) receives the stored normalised activations,
// Xt (optional, bf16) q/gamma, rstd (optional) the per-token reciprocal RMS.  Rows of up to 16*64 16-byte
// vectors (8 for the backward).  nw > 0: nw further workgroups leave the first stage of W's statistics in partials.
int pq_launch_rmsnorm_quant(const void* X, const void* gain, int dtype, int T, int K, float eps, void* Xn, int8_t* Xq,
                            float* gamma, uint16_t* Xt, float* rstd, hipStream_t s, const void* W = nullptr, size_t w_elems = 0,
                            double* partials = nullptr, int nw = 0);
size_t pq_rmsnorm_bwd_scratch_bytes(int T, int K);
int pq_launch_rmsnorm_bwd(const void* dXn, const void* X, const void* gain, const float* rstd, int dtype, int T, int K, void* dX,
                          float* dgain, float* part, hipStream_t s);
// The library's static device scratch (for entry points that must not allocate): its size, and its address on the
// current device (looked up once per device).
size_t pq_static_scratch_bytes();
int pq_static_scratch(void** out);
// Weight statistics, stage 1: per-block fp64 partial sums {sum W, sum |W|}.
int pq_stats_blocks(size_t n_elems);
// dtype: of W and X.  slabs != nullptr: `splits` fp32 slabs [M][N] of a deferred split contraction are summed in slab order into the bf16
// matrix C [M][ldc] by further workgroups of the same launch (N % 8 == 0)
int pq_launch_wstats_quant(const void* W, int dtype, size_t n_elems, double* partials, int nblocks, const void* X, int T, int K,
                           int8_t* Xq, float* gamma, uint16_t* Xt, hipStream_t s, const float* slabs = nullptr, int splits = 0,
                           int M = 0, int N = 0, void* C = nullptr, int ldc = 0);
int pq_launch_wstats_partial(const void* W, int dtype, size_t n_elems, double* partials, int nblocks,
                             hipStream_t s);
// Stage 2 + binarise + pack (both orientations).  Every block re-reduces the partials in the
// same order, block 0 writes mu_lambda.
int pq_launch_pack(const void* W, int dtype, int N, int K, const double* partials, int nblocks,
                   uint32_t* P, uint32_t* Pt, float* mu_lambda, hipStream_t s);
// The weight side of an FFN forward (bf16): stage 1 of three weights' statistics (w[i].partials, w[i].nblocks =
// pq_stats_blocks), the quantiser of X (T rows of D; T may be 0), and the expert rows [Up_e; Gate_e] as one [E][2 r][D]
// matrix: copied to UG, or with UGQ set (INT8 experts) quantised to UGQ / gUG / UGT, with the E * D rows of Down to DownQ /
// gDown / DownT; then the packing of the three.
struct pq_router_job { const void* Wr; int E, k; int* idx; float *gate, *probs; int* hist; };   // (Wr NULL: none)
// The slots of a routed call in expert order, from the router's counts, and their rows in that order (pq_quant.hip).
struct pq_place {
  const int* hist;              // [nblk][E], of `tokens` tokens each
  int nblk, tokens, T, k, E, d;
  const int* idx;
  int *counts, *offsets, *perm, *inv;
  const uint16_t* src;          // [T][d] bf16
  uint16_t* dst;                // [T k][d]
  const int8_t* codes;          // INT8 experts (otherwise NULL): codes [T][d] and gammas [T] go along
  const float* gamma;
  int8_t* codes_out;
  float* gamma_out;
};
int pq_router_tokens(int E);    // tokens per row of hist
struct pq_weight_job { const void* W; int N, K; double* partials; int nblocks; uint32_t* P; uint32_t* Pt; float* mu_lambda; };
struct pq_ffn_prep {
  pq_weight_job w[3];
  const void* X; int T, D; int8_t* Xq; float* gamma; uint16_t* Xt;
  const void *Up, *Gate, *Down; int E, r;
  void* UG;
  int8_t* UGQ; float* gUG; uint16_t* UGT;
  int8_t* DownQ; float* gDown; uint16_t* DownT;
  pq_router_job route;          // (where pq_wstats_quant_router_applies)
};
int pq_launch_ffn_prep(const pq_ffn_prep& p, hipStream_t s);
int pq_launch_pack3(const pq_weight_job* w, const pq_place* place, hipStream_t s);   // place may be NULL
// pq_launch_pack of a bf16 weight (N, K multiples of 32; W NULL: no weight) with the ordering of the slots in the launch
int pq_launch_pack_place(const void* W, int N, int K, const double* partials, int nblocks, uint32_t* P, uint32_t* Pt, float* mu_lambda,
                         const pq_place& place, hipStream_t s);
// pq_launch_wstats_quant (bf16) with the router in the launch
bool pq_wstats_quant_router_applies(int E, int K, long blocks);   // blocks: workgroups of the launch without it
int pq_launch_wstats_quant_router(const void* W, size_t n_elems, double* partials, int nblocks, const void* X, int T, int K, int8_t* Xq, float* gamma,
                                  uint16_t* Xt, const pq_router_job& r, hipStream_t s);
// pq_launch_pack of a bf16 weight (N, K multiples of 32) with the AbsMax quantiser of the rows of two more bf16 matrices in the launch
struct pq_quant_rows_job { const void* src; int rows, cols; int8_t* codes; float* gamma; uint16_t* deq; };
int pq_launch_pack_quant_rows(const void* W, int N, int K, const double* partials, int nblocks, uint32_t* P, uint32_t* Pt, float* mu_lambda,
                              const pq_quant_rows_job* jobs, hipStream_t s);
int pq_launch_router(const void* X, const void* Wr, int dtype, int T, int K, int E, int k, int* idx,
                     float* gate, float* probs, hipStream_t s, int* hist = nullptr);
// two sums of partials in one launch: out[0] = factor [* *dev_factor] * sum(partials[0..n))
int pq_launch_reduce_partials2(const double* pa, int na, float fa, const float* dfa, float* oa, const double* pb, int nb, float fb,
                               const float* dfb, float* ob, hipStream_t s);

// ---- pq_gemm.hip --------------------------------------------------------------------------
enum pq_src_kind {
  PQ_SRC_KC16 = 0,   // bf16, contraction index contiguous: elem(row,k) = p[row*ld + k]
  PQ_SRC_KS16 = 1,   // bf16, contraction index strided:   elem(row,k) = p[k*ld + row]
  PQ_SRC_KC8 = 2,    // int8, contraction contiguous
  PQ_SRC_BITS8 = 3,  // +/-1 as int8 from packed bits, ld = bytes per row
  PQ_SRC_BITS16 = 4, // +/-1 as bf16 from packed bits, ld = bytes per row
  // fp32 I/O only (pq_ref.hip):
  PQ_SRC_KC32 = 5,   // fp32, contraction contiguous
  PQ_SRC_KS32 = 6,   // fp32, contraction strided
  PQ_SRC_KS8 = 7,    // int8, contraction strided
  PQ_SRC_BITSF = 8   // +/-1 from packed bits as a real number
};

struct pq_operand {
  const void* p;
  long ld;             // leading dimension in elements (bytes per row for the BITS kinds)
  int kind;
  const float* kdiv;   // optional: divide element by kdiv[k] (per contraction index); fp32 I/O only
};

enum pq_out_kind { PQ_OUT_F32 = 0, PQ_OUT_BF16 = 1, PQ_OUT_I32 = 2 };

struct pq_epilogue {
  void* C;                    // [M][ldc]
  long ldc;
  int out_kind;
  int accumulate;             // C = C + value
  float scale;                // value = scale * acc, or (scale / row_div[m]) * acc
  const float* dev_scale;     // optional device scalar multiplied into `scale` first (fp32 product)
  const float* row_div;       // optional per-row divisor (gamma_t)
  const float* col_div;       // optional per-column divisor applied after the row scale: value / col_div[n]
  int defer_reduce;           // a split contraction leaves its fp32 slabs in the scratch and launches no reduction: the
                              // caller sums them itself (plain epilogues only, see pq_slab_sum_bf16_body)
  int split_int8;             // int8 GEMM: the contraction may be split (int32 slabs summed exactly); callers that set it
                              // size their scratch with pq_plan_gemm(..., int8 = true, split_int8 = true)
  // optional fixed-order partial reductions, one double per block:
  const void* dot_comp;       // sum_{m,n} comp[m][n] * acc   (comp of the io dtype)
  long ld_comp;
  int comp_kind;              // PQ_OUT_F32 / PQ_OUT_BF16
  const uint8_t* sign_bytes;  // sum_{m,n} (+/-1 from bit n of packed row m) * acc
  long ld_sign;               // bytes per packed row
  double* partials;
  // optional STE clipping mask on the stored value: keep iff |W[m][n] - mu| <= tau
  const void* maskW;
  int mask_kind;              // PQ_OUT_F32 / PQ_OUT_BF16
  const float* mu_dev;        // device pointer to mu
  float tau;
  // optional store limits for outputs narrower than the computed tile range (padded widths): rows >= m_limit and
  // columns >= n_limit are computed but not stored (0 = no limit; n_limit % 4 == 0; plain stores only: no
  // accumulate, mask or dot_comp, whose loads would run past a row's end)
  int m_limit, n_limit;
  // optional second destination: of every 2 * m_split rows the first m_split go to C, the others to C2 (both with their rows
  // closed up): the gradients of matrices that are multiplied as one.  fp32, plain stores only.
  // m_split == 0 (int8 x int8, bf16 outputs that accumulate): C2 [M][ldc] receives the value itself and C then adds c2_scale times it.
  void* C2;
  int m_split;
  float c2_scale;
};

// Optional second contraction accumulated into the same output tile (the rank-r branch fused into
// the 1-bit GEMM): after the main contraction acc1, the accumulator becomes
//     acc = (scale1 * [*dev_scale1] / [row_div1[m]]) * acc1 + sum_{k<K2} A2(m,k) * B2(n,k)
// and the epilogue then applies its own scale.  bf16 operands (KC16 x KC16 or KC16 x KS16).
struct pq_phase2 {
  pq_operand A2, B2;
  int K2;                    // 0 = no second contraction
  float scale1;
  const float* dev_scale1;
  const float* row_div1;
};

// C[M][N] (+)= epilogue( sum_k A(m,k) * B(n,k) ) on the MFMA engine (bf16 or int8 operands).
// Grouped execution over expert segments (Sec. 3.3): `offsets` [n_groups+1] is a device array of
// slot positions.  mode 1: rows [offsets[e], offsets[e+1]) of A and C belong to group e and use
// B + e*b_stride (elements of B's type) -- the per-expert GEMMs of the forward pass;  mode 2: the
// contraction index runs over [offsets[e], offsets[e+1]) and the result goes to C + e*c_stride
// (elements of C's type) -- the per-expert weight gradients.  max_rows bounds a segment (launch size).
// mode 3: two independent GEMMs of the same operand kinds, tile shape and contraction split in one launch;
// workgroups with blockIdx.z == 1 work on the second (plain epilogue: C = scale * acc, or raw slabs when split).  Its
// description is an argument of the paired kernels only.
struct pq_gemm_second {
  pq_operand A, B;
  void* C;
  int ldc;
  float scale;
  float* part;       // split slabs of the second problem
  const float* dev_scale;
  int M, N, nbn;
};
struct pq_gemm_group {
  const int* offsets;
  int n_groups;
  int mode;          // 0 = not grouped
  long b_stride;
  long c_stride;
  int max_rows;
  long coldiv_stride;  // mode 1: group e divides its columns by col_div[e * coldiv_stride + n] (per-expert weight-row scales)
};

// A section of the caller's workspace that a split contraction leaves its slabs in.  Every launch compares what its plan
// writes with `bytes` and is refused (PQ_ERR_WORKSPACE) when the section is too small for it.
struct pq_scratch {
  void* p;
  size_t bytes;
};

struct pq_gemm_plan {
  int bm, bn;        // tile: 64x64, 128x128, 256x256; 128x256 (packed signs, instead of the last), 192x256 (weight gradients)
  int splits;        // contraction splits (1 = none)
  int kchunk;        // contraction elements per split
  int red_blocks;    // number of per-block partial sums written when a reduction is requested
  size_t ws_bytes;   // scratch for the split slabs
  double us;         // the time that the choice expects
};
// what decides between tiles of 256 columns: packed signs in B (the 1-bit forward with int8, dX without), or contraction-strided
// operands on both sides with one destination (weight gradients)
enum pq_plan_kind { PQ_PLAN_ANY = 0, PQ_PLAN_SIGNS = 1, PQ_PLAN_WGRAD = 2 };
pq_gemm_plan pq_plan_gemm(int M, int N, int K, bool int8 = false, bool split_int8 = false, pq_plan_kind kind = PQ_PLAN_ANY);
// whether a second contraction (pq_phase2) can be fused into a GEMM of this plan
inline bool pq_plan_fuses(const pq_gemm_plan& pl) { return pl.splits == 1 || pl.bn < 256; }
// tn: the streaming pair kernel; apart: a launch each; otherwise 64x64 tiles.  ws0, ws1: scratch of the two problems.
struct pq_pair_plan { bool tn, apart; int splits, kchunk; size_t ws0, ws1; };
pq_pair_plan pq_plan_pair(int K, int M0, int N0, int M1, int N1);
// Scratch a grouped launch over contraction ranges (mode 2; M x N per group, total_k indices over all groups) may use
size_t pq_mode2_ws_bytes(int M, int N, int n_groups, int total_k);
// C[M][128] = scale * A B^T for bf16 operands and many rows (the hidden state of the dense high-precision branch
// and its gradient, Sec. 3.2): one workgroup per 32 rows runs the whole contraction through a ring of seven stages of
// direct-to-LDS loads, so nothing is split or reduced.  B is contraction-contiguous or contraction-strided; the
// epilogue may carry dot_comp / partials (one partial sum per workgroup: pq_skinny_blocks(M) of them).
// `applies` states the shapes, alignments and epilogues it takes.
bool pq_skinny_applies(int M, int N, int K, const pq_operand& A, const pq_operand& B, const pq_epilogue& e);
int pq_skinny_blocks(int M);
int pq_launch_skinny(int M, int K, const pq_operand& A, const pq_operand& B, const pq_epilogue& e, hipStream_t s, int prof_label);

// Two bf16 GEMMs with contraction-strided operands on both sides (the rank-r weight gradients dA and dB), in one launch where
// pq_plan_pair finds that better.  Both have plain epilogues: C (fp32) = scale * acc.
// along (may be NULL): the rest of a linear's backward behind dH, which goes before them or in their launch: dW (the same kinds and
// contraction) and, if has_x, dX with the branch's share as its second contraction.
int pq_launch_gemm_pair_ks16(int K, int M0, int N0, const pq_operand& A0, const pq_operand& B0, float* C0, int ldc0, float scale0,
                             int M1, int N1, const pq_operand& A1, const pq_operand& B1, float* C1, int ldc1, float scale1,
                             hipStream_t s, int prof_label0, int prof_label1, pq_scratch sk0, pq_scratch sk1,
                             const pq_reduce_job* jobs = nullptr, bool* jobs_done = nullptr,   // jobs: two scalar reductions to ride along
                             const struct pq_grads* along = nullptr);
// ---- pq_tile.hip: the 64x64 and 128x128 streaming tiles (pl.bm; the contraction split is the caller's plan) ----
int pq_launch_tile(const pq_gemm_plan& pl, int M, int N, int K, const pq_operand& A, const pq_operand& B, const pq_epilogue& epi, hipStream_t s,
                   float* part, const pq_gemm_group& grp, const pq_phase2& ph2, const pq_gemm_second* second = nullptr);
// dHd [M][N] = scale [* *dev_scale] * A B^T, rounded to bf16, straight into dU and dG of the gated unit Hd = silu(G) U (all [M][N] bf16, columns
// from Fv on written as zeros)
struct pq_gemm_act { const void *U, *G; void *dU, *dG; int Fv; };
bool pq_gemm_swiglu_applies(int M, int N, int K);
int pq_launch_gemm_swiglu(int M, int N, int K, const pq_operand& A, const pq_operand& B, float scale, const float* dev_scale, const pq_gemm_act& act,
                          hipStream_t s, int prof_label);
// a product as its launch takes it
struct pq_tile_call {
  int M, N, K;
  pq_operand A, B;
  pq_epilogue epi;
  pq_gemm_group grp;
  pq_gemm_plan pl;
  float* part;
};
bool pq_tile_set_applies(const pq_tile_call* w, int nw, const pq_tile_call* x);   // (x may be NULL)
// 64x64 tiles: three products of contraction-strided operands (split ones leave slabs) and, with x, one of packed signs with a second contraction
int pq_launch_tile_grads(const pq_tile_call (&c)[3], const pq_tile_call* x, const pq_phase2* p2, hipStream_t s);
int pq_launch_tile_set(const pq_tile_call* w, int nw, const pq_tile_call* x, hipStream_t s);
// Products that do not depend on each other: up to four weight gradients and, with has_x, at the end one of a contraction-contiguous
// operand with signs or a contraction-strided one.  One launch where they all take small tiles and their slabs fit side by side
// in the scratch, otherwise one after the other.
struct pq_gemm_call {
  int M, N, K;
  pq_operand A, B;
  pq_epilogue epi;
  const pq_gemm_group* grp;
  int prof_label;
};
struct pq_grads {
  pq_gemm_call w, x;
  pq_phase2 p2;
  bool has_x;
  pq_scratch sk;
};
int pq_launch_gemm_set(const pq_gemm_call* c, int n, hipStream_t s, pq_scratch sk, bool has_x = true);
bool pq_gemm_set_shares(const pq_gemm_call* c, int n, pq_scratch sk, bool has_x);   // (in one launch)
pq_gemm_plan pq_plan_dual(int M, int N, int K, bool int8);   // (its ws_bytes: the slabs of both)
int pq_launch_gemm_dual(int M, int N, int K, const pq_operand& A0, const pq_operand& B0, const pq_epilogue& e0, const pq_operand& A1,
                        const pq_operand& B1, void* C1, const float* dev_scale1, hipStream_t s, int prof_label, pq_scratch sk);
int pq_launch_gemm(int M, int N, int K, const pq_operand& A, const pq_operand& B,
                   const pq_epilogue& epi, hipStream_t s, int prof_label = PQP_GEMM_OTHER,
                   pq_scratch sk = {nullptr, 0}, const pq_gemm_group* group = nullptr,
                   const pq_phase2* phase2 = nullptr);

// ---- pq_ref.hip ---------------------------------------------------------------------------
// Reference-precision products (fp32 I/O): fp64 products and sums, C fp32.  `form` names the operand kinds.
enum pq_ref_form {
  PQ_REF_CC = 0,      // A KC32, B KC32
  PQ_REF_CS = 1,      // A KC32, B KS32
  PQ_REF_CBITS = 2,   // A KC32, B packed signs; then, K2 > 0, a second contraction A2 (KC32) x B2 (KS32) into the same sums:
                      // (scale1 [* *dev_scale1]) * sum_k A B + sum_k2 A2 B2
  PQ_REF_SS8 = 3,     // A KS32, B KS8 divided by its kdiv
  PQ_REF_SS = 4,      // A KS32, B KS32
  // the same with the first contraction already done in fixed point (pq_fixed.hip): its sums are read from `sums` and A, B are
  // looked at only for tiles with rows that are not finite or sums that their elements' range leaves out
  PQ_REF_SUM_CBITS = 5,
  PQ_REF_SUM_SS8 = 6
};
struct pq_ref_problem {
  int form, M, N, K, K2, cfg;   // cfg is set by the launcher
  pq_operand A, B, A2, B2;
  float scale1;
  const float* dev_scale1;
  const double* sums;           // SUM forms: [M][N] sums of the digit products
  const int* exps;              // ... and the rows' exponents
  const int* counts;            // SUM_SS8: [2 M + N], what decides whether a sum of digits may be taken (pq_fixed.hip)
  pq_epilogue epi;              // scale, dev_scale, accumulate, dot_comp, sign_bytes, partials and the clip mask; C is fp32
};
constexpr int PQ_REF_MAX = 3;
int pq_ref_red_blocks(int M, int N, int K);   // partial sums one product leaves when its epilogue asks for them (SUM forms: K = -1)
// Up to PQ_REF_MAX independent products in one launch per tile class (at most two launches); up to two scalar reductions of
// partials that EARLIER launches left ride along.
int pq_launch_ref(pq_ref_problem* p, int n, const pq_reduce_job* jobs, int njobs, hipStream_t s, int prof_label);
// One product (form CC) and the packing of an fp32 weight [N][K] in one launch, where the product is small enough to share it.
bool pq_ref_rides(int M, int N, int K);
int pq_launch_ref_pack(const pq_ref_problem& p, const float* W, int N, int K, const double* partials, int nparts, uint32_t* P, uint32_t* Pt,
                       float* mu_lambda, hipStream_t s);
// Y [T][N] = (beta lambda / gamma_t) * Xq P^T + alpha * H B^T in one launch (H [T][r], B [N][r] fp32 as KC32 operands).
struct pq_ref_linear {
  const int8_t* Xq;             // [T][K]
  const uint32_t* P;            // [N][K/32]
  const float *lambda, *gamma;
  pq_operand H, B;
  float* Y;
  int T, N, K, r;
  float alpha, beta;
};
bool pq_ref_linear_applies(int T, int N, int K);
int pq_launch_ref_linear(const pq_ref_linear& p, hipStream_t s);

// ---- pq_fixed.hip -------------------------------------------------------------------------
// Fixed-point form of dY for the two large contractions of the fp32 backward: digits Drow of dY's rows with exponents rexp [T], digits
// Dcol of the columns of dY / gamma with exponents cexp [N], the codes transposed (qT) and the signs as bytes (from Pt [K][N/32]), each in
// the tiles that the products stream (pq_fixed.hip): rows rounded up to whole panels, PQ_FIXED_M of digits, PQ_FIXED_N of signs and codes,
// the contraction to whole 64.  colmax: [pq_fixed_max_rows(T)][N] words of scratch.  counts [2 N + K]: small and zero elements of the
// columns, zero codes of the channels.
constexpr int PQ_FIXED_DIGITS = 7;
constexpr int PQ_FIXED_M = 64, PQ_FIXED_N = 128;
constexpr int PQ_FIXED_NOT_FINITE = 1 << 20;         // the exponent of a row with infinities or NaN (its digits are zero)
int pq_fixed_max_rows(int T);
int pq_launch_fixed_split(const float* dY, const float* gamma, const int8_t* q, int T, int N, int K, int8_t* Drow, int* rexp, int8_t* Dcol,
                          int* cexp, int8_t* qT, uint32_t* colmax, int* counts, const uint32_t* Pt, int8_t* signs, hipStream_t s);
// SX [T][K] = dY S and SW [N][K] = (dY / gamma)^T q from those digits
int pq_launch_fixed_products(const int8_t* Drow, const int* rexp, const int8_t* signs, double* SX, const int8_t* Dcol, const int* cexp, const int8_t* qT,
                             double* SW, int T, int N, int K, hipStream_t s);

// ---- pq_decode.hip ------------------------------------------------------------------------
size_t pq_decode_ws_layout(const pq_decode_desc& d, size_t* off);
int pq_launch_decode(const pq_decode_desc& d, const void* X, const uint32_t* packed, const uint16_t* scale_fp16,
                     const void* hpA, const void* hpB, const void* Wr, void* Y, int32_t* acc_out, void* workspace,
                     hipStream_t s, const float* gA = nullptr, const float* gB = nullptr);
int pq_launch_retile64(const uint32_t* packed, int N, int K, uint32_t* tiled, hipStream_t s);
int pq_launch_decode_ffn(int L, int B, int D, int F, int r, int E, int topk, float alpha, const void* X, const uint32_t* packed_upgate,
                         const uint16_t* scale_upgate, const uint32_t* packed_down, const uint16_t* scale_down,
                         const void* UpGate, const void* Down, const void* Wr, void* Y, int32_t* acc_upgate, void* UG,
                         void* ws1, void* ws2, float* amax_part, hipStream_t s);   // amax_part: [L][B][8] floats of scratch, [L][ceil(F/64)] for one token

// ---- pq_moe.hip ---------------------------------------------------------------------------
int pq_launch_gather_rows(const void* src, const int* perm, int k, int S, int d, void* dst, hipStream_t s);
int pq_launch_swiglu_quant(const void* U, const void* G, int T, int F, int Fv, int8_t* Hq, float* gamma, void* Ht, hipStream_t s);
int pq_launch_swiglu_bwd(const void* dHd, const void* U, const void* G, int T, int F, int Fv, void* dU, void* dG, hipStream_t s);
// ue, ge (and du, dg) have a row stride of ld elements: r, or 2 r when both lie side by side in one [S][2 r] matrix
// (INT8 experts: with the quantiser of its rows, of up to 2048 elements; at the de-quantised copy)
bool pq_expert_act_quant_applies(int r);
int pq_launch_expert_act_quant(const void* ue, const void* ge, int ld, int S, int r, int8_t* aq, float* gamma, void* at, hipStream_t s);
int pq_launch_expert_act(const void* ue, const void* ge, int ld, int S, int r, void* a, hipStream_t s);
// perm == NULL: a single branch (gate 1).  dWr != NULL: its n_wr elements are cleared and jobs[0..1] reduced in the same launch.
int pq_launch_expert_act_bwd(const void* da, const void* ue, const void* ge, const void* a, const int* perm, const float* gate,
                             float alpha, int S, int r, int ld, void* du, void* dg, void* as, float* dWr, int n_wr,
                             const pq_reduce_job* jobs, hipStream_t s);
int pq_rowdot_blocks(int S);
// rd[pos] = <dY[perm[pos] / k], Ys[pos]>, partial[pq_rowdot_blocks(S)] of sum gate * rd, dst[pos] (may be NULL) = the dY row
// [* alpha * gate]
int pq_launch_slot_grad(const void* dY, const void* Ys, const int* perm, const float* gate, float alpha, bool scale, int k, int S, int d,
                        void* dst, float* rd, double* partial, hipStream_t s);
int pq_launch_combine_fwd(void* Y, const void* Ys, const int* inv, const float* gate, float alpha, int T, int k, int d, hipStream_t s);
size_t pq_dwr_scratch_bytes(int T, int d, int E);
// router backward and dWr: dlogit [T][E] from rd and the softmax, dWr = dlogit^T X.  jobs: two scalar
// reductions of partials that earlier launches left, in the last launch.
int pq_launch_dwr(const float* rd, const int* inv, const int* idx, const float* probs, float alpha, int k, float* dlogit, const void* X, int T,
                  int d, int E, float* part, float* dWr, const pq_reduce_job* jobs, hipStream_t s);
int pq_launch_combine_bwd(void* dX, const void* dXs, const int* inv, const float* dlogit, const void* Wr, int T, int k, int d, int E,
                          hipStream_t s);
int pq_launch_lincomb(void* out, const void* x0, const void* x1, const void* x2, const void* x3, float c0, float c1, float c2,
                      float c3, size_t n, hipStream_t s);
