// C-ABI entry points of libpquant: argument validation, buffer layout, kernel sequencing.
#include <stdarg.h>
#include <stdio.h>
#include <string.h>
#include "pq_internal.h"

static thread_local char g_err[512] = "";

int pq_set_error(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

extern "C" const char* pq_last_error_string(void) { return g_err; }
extern "C" int pq_version(void) { return 100; }

// ---------------------------------------------------------------------------------------------
// Optional per-kernel event timing
// ---------------------------------------------------------------------------------------------
#include <mutex>
#include <vector>
namespace {
struct prof_sample { hipEvent_t a, b; int label; bool closed; };
bool g_prof_on = false;
std::mutex g_prof_mu;
std::vector<prof_sample*> g_prof_samples;
const char* const g_prof_names[PQP_COUNT] = {
    "quant_act", "wstats_partial", "pack_sign", "router", "reduce_partials",
    "gemm_onebit_fwd", "gemm_hp_H", "gemm_hp_Y", "gemm_dH", "gemm_dX", "gemm_dX_hp",
    "gemm_dW", "gemm_dB", "gemm_dA", "gemm_other", "decode_prep", "decode_h", "decode_main", "moe_route", "moe_elementwise", "swiglu", "gemm_expert", "glue", "splitk_reduce", "rmsnorm_quant", "rmsnorm_bwd"};
}  // namespace

pq_prof_scope::pq_prof_scope(int label_, hipStream_t s_) : label(label_), s(s_), slot(nullptr) {
  if (!g_prof_on) return;
  prof_sample* ps = new prof_sample{nullptr, nullptr, label_, false};
  if (hipEventCreate(&ps->a) != hipSuccess || hipEventCreate(&ps->b) != hipSuccess) { delete ps; return; }
  (void)hipEventRecord(ps->a, s);
  slot = ps;
}
pq_prof_scope::~pq_prof_scope() {
  if (!slot) return;
  prof_sample* ps = (prof_sample*)slot;
  (void)hipEventRecord(ps->b, s);
  ps->closed = true;
  std::lock_guard<std::mutex> g(g_prof_mu);
  g_prof_samples.push_back(ps);
}

extern "C" int pq_prof_enable(int on) { g_prof_on = on != 0; return PQ_OK; }
extern "C" int pq_prof_count(void) { return PQP_COUNT; }
extern "C" const char* pq_prof_label(int label) { return (label >= 0 && label < PQP_COUNT) ? g_prof_names[label] : ""; }
extern "C" int pq_prof_read(int label, double* total_ms, int* launches) {
  if (!total_ms || !launches) return pq_set_error(PQ_ERR_BAD_ARG, "NULL output");
  std::lock_guard<std::mutex> g(g_prof_mu);
  double tot = 0.0; int n = 0;
  for (prof_sample* ps : g_prof_samples) {
    if (ps->label != label || !ps->closed) continue;
    float ms = 0.f;
    PQ_CHECK_HIP(hipEventSynchronize(ps->b));
    PQ_CHECK_HIP(hipEventElapsedTime(&ms, ps->a, ps->b));
    tot += ms; ++n;
  }
  *total_ms = tot; *launches = n;
  return PQ_OK;
}
extern "C" int pq_prof_reset(void) {
  std::lock_guard<std::mutex> g(g_prof_mu);
  for (prof_sample* ps : g_prof_samples) { (void)hipEventDestroy(ps->a); (void)hipEventDestroy(ps->b); delete ps; }
  g_prof_samples.clear();
  return PQ_OK;
}

namespace {

inline bool aligned16(const void* p) { return (((uintptr_t)p) & 15u) == 0; }
inline size_t esize(int dtype) { return dtype == PQ_BF16 ? 2 : 4; }
inline int out_kind_of(int dtype) { return dtype == PQ_BF16 ? PQ_OUT_BF16 : PQ_OUT_F32; }

#define PQ_REQUIRE(cond, code, ...) \
  do { if (!(cond)) return pq_set_error(code, __VA_ARGS__); } while (0)

int check_dtype(int dtype) {
  PQ_REQUIRE(dtype == PQ_F32 || dtype == PQ_BF16, PQ_ERR_DTYPE, "dtype %d is not PQ_F32 or PQ_BF16", dtype);
  return PQ_OK;
}

pq_epilogue epi_zero() {
  pq_epilogue e;
  memset(&e, 0, sizeof(e));
  e.scale = 1.0f;
  return e;
}

pq_ref_problem ref_problem(int form, int M, int N, int K, const pq_operand& A, const pq_operand& B, const pq_epilogue& e) {
  pq_ref_problem p;
  memset(&p, 0, sizeof(p));
  p.form = form; p.M = M; p.N = N; p.K = K; p.A = A; p.B = B; p.epi = e;
  return p;
}

// Buffer layout of one linear.  Sections are 256-byte aligned.
struct lin_layout {
  // ctx (saved by forward for backward)
  size_t mulam, P, Pt, Xq, gamma, Xt, H, ctx_total;
  // routed experts (n_experts > 1): routing decisions, the permuted activations, per-slot hidden states and outputs
  size_t idx, gate, probs, counts, offsets, perm, inv, Xp, Hs, Ys;
  // INT8 form of the dense branch: the ctx of pq_hp_int8_* behind the linear's own
  size_t hp8, hp8_bytes;
  // workspace (scratch)
  size_t stat_partials, red_a, red_b, dH, w_Xq, w_gamma, w_H, splitk, splitk2, splitk_bytes, splitk2_bytes, ws_base, ws_total;
  size_t hist, dYp, rd, dHs, dXs, dlogit, dwr, hp8_ws, hp8_ws_bytes;
  // fp32 I/O in fixed point (pq_fixed.hip): a region of fx_bytes (0: the call has none) behind everything else, which only a backward
  // uses, and only if the workspace holds it
  size_t fx_drow, fx_rexp, fx_dcol, fx_cexp, fx_qT, fx_colmax, fx_counts, fx_red_b, fx_signs, fx_SW, fx_SX, fx_bytes;
  int n_red_a, n_red_b;
};

struct cursor {
  size_t off = 0;
  size_t take(size_t bytes) {
    size_t o = off;
    off = pq_align_up(off + bytes, 256);
    return o;
  }
};

// The two large contractions of the fp32 backward in fixed point: seven int8 products of one in fp64, a quarter of its time, but four
// more launches (some 20 us), 8 bytes of sums per output and 22 of digits per element of dY, written and read.  The line was drawn while an
// output's seven int32 sums went through memory (56 bytes: its terms in 1 / tokens and 1 / d_out) and has not been moved since.
// Backward against the fp64 products, both as they are now, 40 shapes of 64 to 65536 tokens and widths of 128 to 11008: inside the line 1.11 x
// (65536 tokens 512->512) to 3.95 x (4096 4096->11008), 2048 tokens 2048x2048 554 / 168 us; outside it 0.52 x (512 512->512, 32768 256->256) to
// 1.9 x: the digits would be ahead for few tokens through wide layers (256 11008->4096 770 / 405 us, 128 8192->8192 593 / 514) and narrow outputs of
// few thousand tokens (2048 4096->256 165 / 99), behind for 64 tokens (8192->8192 349 / 503) and many tokens through narrow layers.
// The int32 sums of dW hold tokens * 2^14, those of dX d_out * 2^7.  Calls whose region would take more than FIXED_MAX_BYTES keep the fp64
// products.  The region is counted as 14 tokens * d_out + tokens * d_in + 28 d_in * max(tokens, d_out) bytes, what it was with the int32 sums and callers
// have sized it by: 172 MiB at 2048 tokens 2048x2048 (130 used), 1.8 GiB at 4096 tokens 4096x11008 (1.1 used); the 1.9 GiB that
// 8192 tokens 4096->11008 would use count as 2.4.
constexpr size_t FIXED_MAX_BYTES = (size_t)2 << 30;
bool fixed_applies(int T, int K, int N) {
  return T <= 65536 && N <= 65536 && (double)T * K * N >= 1.2e9 && 1.0 / T + 1.0 / N + 0.4 / K <= 1.0 / 320;
}

lin_layout make_layout(const pq_linear_desc& d) {
  lin_layout L;
  memset(&L, 0, sizeof(L));
  const bool routed = d.n_experts > 1 && d.hp_rank > 0;
  const bool hp8 = d.hp_kind == PQ_HP_LOWRANK_INT8 && d.hp_rank > 0;
  // the dense-branch sections (H, dH, the rank-r GEMM plans) are sized for the dense branch only
  const size_t T = d.tokens, K = d.d_in, N = d.d_out, r = (routed || hp8) ? 0 : d.hp_rank, es = esize(d.io_dtype);
  const bool bf16 = d.io_dtype == PQ_BF16;   // fp32 I/O: reference-precision products, nothing is split
  cursor c;
  L.mulam = c.take(2 * sizeof(float));
  L.P = c.take(N * K / 8);
  L.Pt = c.take(N * K / 8);
  L.Xq = c.take(T * K);
  L.gamma = c.take(T * sizeof(float));
  L.Xt = c.take(d.io_dtype == PQ_BF16 ? T * K * 2 : 0);
  L.H = c.take(T * r * es);
  const size_t S = T * (size_t)d.top_k, E = d.n_experts, re = d.hp_rank;
  if (routed) {
    L.idx = c.take(S * 4); L.gate = c.take(S * 4); L.probs = c.take(T * E * 4);
    L.counts = c.take(E * 4); L.offsets = c.take((E + 1) * 4); L.perm = c.take(S * 4); L.inv = c.take(S * 4);
    L.Xp = c.take(S * K * 2); L.Hs = c.take(S * re * 2); L.Ys = c.take(S * N * 2);
  }
  if (hp8) {
    L.hp8_bytes = pq_hp_int8_ctx_bytes(d.tokens, d.d_in, d.d_out, d.hp_rank);
    L.hp8 = c.take(L.hp8_bytes);
  }
  L.ctx_total = c.off > 0 ? c.off : 256;
  cursor w;
  L.stat_partials = w.take(2 * sizeof(double) * 1024);
  const int Ti = d.tokens, Ki = d.d_in, Ni = d.d_out, ri = (int)r;
  L.n_red_a = r ? (bf16 ? pq_plan_gemm(Ti, ri, Ni).red_blocks : pq_ref_red_blocks(Ti, ri, Ni)) : 0;   // dH GEMM
  if (r && pq_skinny_blocks(Ti) > L.n_red_a) L.n_red_a = pq_skinny_blocks(Ti);   // room for the streaming rank-r kernel's partials
  L.n_red_b = bf16 ? pq_plan_gemm(Ni, Ki, Ti, false, false, PQ_PLAN_WGRAD).red_blocks : pq_ref_red_blocks(Ni, Ki, Ti);              // dW GEMM
  size_t sk = 0;
  const int shapes[7][3] = {{Ti, ri, Ki}, {Ti, Ni, ri}, {Ti, ri, Ni}, {Ti, Ki, ri}, {Ni, Ki, Ti}, {Ni, ri, Ti}, {ri, Ki, Ti}};
  for (const auto& sh : shapes) {
    if (!bf16 || sh[0] <= 0 || sh[1] <= 0) continue;
    const size_t b = pq_plan_gemm(sh[0], sh[1], sh[2]).ws_bytes;
    if (b > sk) sk = b;
  }
  if (bf16) {   // the products with packed signs (forward and dX) and the paired factor gradients
    const size_t f = pq_plan_gemm(Ti, Ni, Ki, true, true, PQ_PLAN_SIGNS).ws_bytes,
                 x = pq_plan_gemm(Ti, Ki, Ni, false, false, PQ_PLAN_SIGNS).ws_bytes;
    if (Ti > 0 && f > sk) sk = f;
    if (Ti > 0 && x > sk) sk = x;
    if (ri > 0 && pq_plan_pair(Ti, Ni, ri, ri, Ki).ws0 > sk) sk = pq_plan_pair(Ti, Ni, ri, ri, Ki).ws0;
  }
  if (routed) {
    L.n_red_a = pq_rowdot_blocks((int)S);
    if (8 * S * re * sizeof(float) > sk) sk = 8 * S * re * sizeof(float);   // narrow grouped GEMMs split the contraction up to 8 ways
    // so do the per-expert factor gradients over their slot ranges
    if (pq_mode2_ws_bytes(Ni, (int)re, d.n_experts, (int)S) > sk) sk = pq_mode2_ws_bytes(Ni, (int)re, d.n_experts, (int)S);
    if (pq_mode2_ws_bytes((int)re, Ki, d.n_experts, (int)S) > sk) sk = pq_mode2_ws_bytes((int)re, Ki, d.n_experts, (int)S);
  }
  if (hp8) L.n_red_a = pq_plan_gemm(Ti, d.hp_rank, Ni).red_blocks;      // the INT8 branch's dH GEMM leaves the partials of d alpha
  L.red_a = w.take(sizeof(double) * (size_t)(L.n_red_a > 0 ? L.n_red_a : 1));
  L.red_b = w.take(sizeof(double) * (size_t)L.n_red_b);
  L.dH = w.take(T * r * es);
  L.w_Xq = w.take(T * K);          // used when forward runs without a ctx (inference)
  L.w_gamma = w.take(T * sizeof(float));
  L.w_H = w.take(T * r * es);
  L.splitk = w.take(sk);
  L.splitk_bytes = sk;
  // slabs of dA, which shares a launch with dB (whose slabs are in the region above)
  const size_t sk2a = (bf16 && ri > 0) ? pq_plan_gemm(ri, Ki, Ti).ws_bytes : 0, sk2b = (bf16 && ri > 0) ? pq_plan_pair(Ti, Ni, ri, ri, Ki).ws1 : 0;
  L.splitk2_bytes = sk2a > sk2b ? sk2a : sk2b;
  L.splitk2 = w.take(L.splitk2_bytes);
  if (routed) {
    // The router's counts, which the forward alone needs, lie in the backward's dYp: at most E <= 64 bytes a token against 2 k d_out >= 64, so
    // that they add nothing to what a workspace holds.
    const size_t rt = pq_router_tokens((int)E), counts = (T + rt - 1) / rt * E * sizeof(int), dyp = S * N * 2;
    L.hist = L.dYp = w.take(counts > dyp ? counts : dyp);
    L.rd = w.take(S * 4); L.dHs = w.take(S * re * 2); L.dXs = w.take(S * K * 2);
    L.dlogit = w.take(T * E * 4);
    L.dwr = w.take(pq_dwr_scratch_bytes(d.tokens, d.d_in, d.n_experts));
  }
  if (hp8) {
    L.hp8_ws_bytes = pq_hp_int8_workspace_bytes(d.tokens, d.d_in, d.d_out, d.hp_rank);
    L.hp8_ws = w.take(L.hp8_ws_bytes);
  }
  L.ws_base = L.ws_total = w.off;
  if (!bf16 && d.w_kind == PQ_W_MASTER && Ni % 32 == 0 && fixed_applies(Ti, Ki, Ni)) {   // (what a backward takes)
    const size_t T64 = pq_align_up(T, 64), N64 = pq_align_up(N, 64), Kp = pq_align_up(K, PQ_FIXED_N);
    cursor x;
    L.fx_drow = x.take(PQ_FIXED_DIGITS * T64 * N64); L.fx_rexp = x.take(T * sizeof(int));
    L.fx_dcol = x.take(PQ_FIXED_DIGITS * N64 * T64); L.fx_cexp = x.take(N * sizeof(int));
    L.fx_qT = x.take(Kp * T64); L.fx_signs = x.take(Kp * N64);
    L.fx_colmax = x.take(pq_fixed_max_rows(Ti) * N * sizeof(uint32_t));
    L.fx_counts = x.take((2 * N + K) * sizeof(int));
    L.fx_red_b = x.take(sizeof(double) * (size_t)pq_ref_red_blocks(Ni, Ki, -1));
    L.fx_SW = x.take(N * K * sizeof(double)); L.fx_SX = x.take(T * K * sizeof(double));
    // (never smaller than what callers have sized it by, see FIXED_MAX_BYTES)
    const size_t least = 14 * T * N + K * T + 28 * K * (T > N ? T : N);
    if (x.off < least) x.take(least - x.off);
    if (x.off <= FIXED_MAX_BYTES) {
      L.fx_bytes = x.off;
      L.ws_total += x.off;
    }
  }
  return L;
}

int check_desc(const pq_linear_desc* d, bool training) {
  PQ_REQUIRE(d != nullptr, PQ_ERR_BAD_ARG, "desc is NULL");
  PQ_REQUIRE(d->tokens >= 0 && d->d_in > 0 && d->d_out > 0 && d->hp_rank >= 0, PQ_ERR_BAD_ARG,
             "negative or zero dimension (tokens=%d d_in=%d d_out=%d hp_rank=%d)", d->tokens, d->d_in,
             d->d_out, d->hp_rank);
  if (int e = check_dtype(d->io_dtype)) return e;
  PQ_REQUIRE(d->w_kind == PQ_W_MASTER || d->w_kind == PQ_W_PACKED, PQ_ERR_BAD_ARG, "unknown w_kind %d", d->w_kind);
  PQ_REQUIRE(d->ste_mode == PQ_STE_IDENTITY || d->ste_mode == PQ_STE_CLIP, PQ_ERR_BAD_ARG, "unknown ste_mode %d", d->ste_mode);
  PQ_REQUIRE(d->d_in % 32 == 0, PQ_ERR_SHAPE, "d_in=%d must be a multiple of 32", d->d_in);
  PQ_REQUIRE(d->d_out % 8 == 0, PQ_ERR_SHAPE, "d_out=%d must be a multiple of 8", d->d_out);
  PQ_REQUIRE(d->hp_rank % 8 == 0, PQ_ERR_SHAPE, "hp_rank=%d must be a multiple of 8", d->hp_rank);
  PQ_REQUIRE(d->n_experts >= 1 && d->n_experts <= 64, PQ_ERR_BAD_ARG, "n_experts=%d must be in 1..64", d->n_experts);
  PQ_REQUIRE(d->top_k >= 1 && d->top_k <= d->n_experts, PQ_ERR_BAD_ARG, "top_k=%d must be in 1..n_experts", d->top_k);
  if (training) {
    PQ_REQUIRE(d->d_out % 32 == 0, PQ_ERR_SHAPE, "training needs d_out=%d to be a multiple of 32", d->d_out);
    PQ_REQUIRE(d->w_kind == PQ_W_MASTER, PQ_ERR_BAD_ARG, "backward needs latent weights (PQ_W_MASTER)");
  }
  PQ_REQUIRE(d->hp_kind == PQ_HP_LOWRANK_BF16 || d->hp_kind == PQ_HP_LOWRANK_INT8, PQ_ERR_BAD_ARG, "unknown hp_kind %d", d->hp_kind);
  if (d->n_experts > 1 && d->hp_rank > 0) {
    PQ_REQUIRE(d->io_dtype == PQ_BF16, PQ_ERR_DTYPE, "routed experts (n_experts=%d) run on bf16 I/O only", d->n_experts);
    PQ_REQUIRE(d->hp_kind == PQ_HP_LOWRANK_BF16, PQ_ERR_BAD_ARG, "routed experts take the 16-bit form of the high-precision branch");
    PQ_REQUIRE(d->d_out % 32 == 0, PQ_ERR_SHAPE, "routed experts need d_out=%d to be a multiple of 32", d->d_out);
  }
  if (d->hp_kind == PQ_HP_LOWRANK_INT8 && d->hp_rank > 0) {
    PQ_REQUIRE(d->io_dtype == PQ_BF16, PQ_ERR_DTYPE, "the INT8 high-precision branch runs on bf16 I/O only");
    PQ_REQUIRE(d->d_out % 32 == 0 && d->hp_rank % 32 == 0, PQ_ERR_SHAPE,
               "the INT8 high-precision branch needs d_out=%d and hp_rank=%d to be multiples of 32", d->d_out, d->hp_rank);
  }
  return PQ_OK;
}

}  // namespace

// ---------------------------------------------------------------------------------------------
extern "C" int pq_quant_act(const void* X, int32_t dtype, int32_t T, int32_t K, int8_t* Xq, float* gamma,
                            void* stream) {
  if (int e = check_dtype(dtype)) return e;
  PQ_REQUIRE(T >= 0 && K > 0, PQ_ERR_BAD_ARG, "bad size T=%d K=%d", T, K);
  PQ_REQUIRE(K % 32 == 0, PQ_ERR_SHAPE, "K=%d must be a multiple of 32", K);
  if (T == 0) return PQ_OK;
  PQ_REQUIRE(X && Xq && gamma, PQ_ERR_BAD_ARG, "NULL buffer");
  PQ_REQUIRE(aligned16(X) && aligned16(Xq), PQ_ERR_SHAPE, "X and Xq must be 16-byte aligned");
  return pq_launch_quant_act(X, dtype, T, K, Xq, gamma, nullptr, (hipStream_t)stream);
}

extern "C" int pq_rmsnorm_quant_fwd(const void* X, const void* gain, int32_t dtype, int32_t T, int32_t K, float eps, void* Xn,
                                    int8_t* Xq, float* gamma, void* Xt, float* rstd, void* stream) {
  if (int e = check_dtype(dtype)) return e;
  PQ_REQUIRE(T >= 0 && K > 0, PQ_ERR_BAD_ARG, "bad size T=%d K=%d", T, K);
  PQ_REQUIRE(K % 32 == 0, PQ_ERR_SHAPE, "K=%d must be a multiple of 32", K);
  PQ_REQUIRE(eps >= 0.0f, PQ_ERR_BAD_ARG, "eps must not be negative");
  PQ_REQUIRE(K <= (dtype == PQ_F32 ? 4096 : 8192), PQ_ERR_SHAPE, "K=%d exceeds the row length this call keeps in registers", K);
  if (T == 0) return PQ_OK;
  PQ_REQUIRE(X && gain && Xq && gamma, PQ_ERR_BAD_ARG, "NULL buffer");
  PQ_REQUIRE(aligned16(X) && aligned16(gain) && aligned16(Xq) && aligned16(Xn) && aligned16(Xt), PQ_ERR_SHAPE,
             "buffers must be 16-byte aligned");
  return pq_launch_rmsnorm_quant(X, gain, dtype, T, K, eps, Xn, Xq, gamma, (uint16_t*)Xt, rstd, (hipStream_t)stream);
}

extern "C" size_t pq_rmsnorm_bwd_workspace_bytes(int32_t T, int32_t K) {
  if (T < 0 || K <= 0) return 0;
  return pq_rmsnorm_bwd_scratch_bytes(T, K) + 256;
}

extern "C" int pq_rmsnorm_bwd(const void* dXn, const void* X, const void* gain, const float* rstd, int32_t dtype, int32_t T,
                              int32_t K, void* dX, float* dgain, void* workspace, size_t workspace_bytes, void* stream) {
  if (int e = check_dtype(dtype)) return e;
  PQ_REQUIRE(T >= 0 && K > 0, PQ_ERR_BAD_ARG, "bad size T=%d K=%d", T, K);
  PQ_REQUIRE(K % 32 == 0, PQ_ERR_SHAPE, "K=%d must be a multiple of 32", K);
  PQ_REQUIRE(K <= (dtype == PQ_F32 ? 2048 : 4096), PQ_ERR_SHAPE, "K=%d exceeds the row length this call keeps in registers", K);
  PQ_REQUIRE(dgain && gain, PQ_ERR_BAD_ARG, "NULL buffer");
  PQ_REQUIRE(T == 0 || (dXn && X && rstd && dX), PQ_ERR_BAD_ARG, "NULL buffer");
  PQ_REQUIRE(aligned16(dXn) && aligned16(X) && aligned16(gain) && aligned16(dX), PQ_ERR_SHAPE, "buffers must be 16-byte aligned");
  PQ_REQUIRE(workspace_bytes >= pq_rmsnorm_bwd_workspace_bytes(T, K), PQ_ERR_WORKSPACE, "workspace too small");
  PQ_REQUIRE(T == 0 || workspace, PQ_ERR_BAD_ARG, "NULL workspace");
  float* part = (float*)(((uintptr_t)workspace + 255) & ~(uintptr_t)255);
  return pq_launch_rmsnorm_bwd(dXn, X, gain, rstd, dtype, T, K, dX, dgain, part, (hipStream_t)stream);
}

extern "C" size_t pq_rmsnorm_bwd_static_max_bytes(void) { return pq_static_scratch_bytes(); }

extern "C" int pq_rmsnorm_bwd_static(const void* dXn, const void* X, const void* gain, const float* rstd, int32_t dtype, int32_t T,
                                     int32_t K, void* dX, float* dgain, void* stream) {
  if (int e = check_dtype(dtype)) return e;
  PQ_REQUIRE(T >= 0 && K > 0, PQ_ERR_BAD_ARG, "bad size T=%d K=%d", T, K);
  PQ_REQUIRE(K % 32 == 0, PQ_ERR_SHAPE, "K=%d must be a multiple of 32", K);
  PQ_REQUIRE(K <= (dtype == PQ_F32 ? 2048 : 4096), PQ_ERR_SHAPE, "K=%d exceeds the row length this call keeps in registers", K);
  PQ_REQUIRE(dgain && gain, PQ_ERR_BAD_ARG, "NULL buffer");
  PQ_REQUIRE(T == 0 || (dXn && X && rstd && dX), PQ_ERR_BAD_ARG, "NULL buffer");
  PQ_REQUIRE(aligned16(dXn) && aligned16(X) && aligned16(gain) && aligned16(dX), PQ_ERR_SHAPE, "buffers must be 16-byte aligned");
  const size_t need = pq_rmsnorm_bwd_scratch_bytes(T, K);
  PQ_REQUIRE(need <= pq_static_scratch_bytes(), PQ_ERR_WORKSPACE,
             "T=%d x K=%d needs %zu bytes of partial rows, the static scratch holds %zu: use pq_rmsnorm_bwd with a workspace",
             T, K, need, pq_static_scratch_bytes());
  void* part = nullptr;
  if (int e = pq_static_scratch(&part)) return e;
  return pq_launch_rmsnorm_bwd(dXn, X, gain, rstd, dtype, T, K, dX, dgain, (float*)part, (hipStream_t)stream);
}

extern "C" size_t pq_pack_workspace_bytes(int32_t N, int32_t K) {
  (void)N; (void)K;
  return 2 * sizeof(double) * 1024;
}

extern "C" int pq_pack_sign(const void* W, int32_t w_dtype, int32_t N, int32_t K, uint32_t* packed,
                            uint32_t* packed_t, float* mu_lambda, void* workspace, size_t workspace_bytes,
                            void* stream) {
  if (int e = check_dtype(w_dtype)) return e;
  PQ_REQUIRE(N > 0 && K > 0, PQ_ERR_BAD_ARG, "bad size N=%d K=%d", N, K);
  PQ_REQUIRE(K % 4 == 0, PQ_ERR_SHAPE, "K=%d must be a multiple of 4", K);
  PQ_REQUIRE(((size_t)N * K) % 8 == 0, PQ_ERR_SHAPE, "N*K=%zu must be a multiple of 8", (size_t)N * K);
  PQ_REQUIRE(W && packed && mu_lambda && workspace, PQ_ERR_BAD_ARG, "NULL buffer");
  PQ_REQUIRE(aligned16(W) && aligned16(workspace), PQ_ERR_SHAPE, "W and workspace must be 16-byte aligned");
  PQ_REQUIRE(workspace_bytes >= pq_pack_workspace_bytes(N, K), PQ_ERR_WORKSPACE, "workspace too small: %zu < %zu",
             workspace_bytes, pq_pack_workspace_bytes(N, K));
  hipStream_t s = (hipStream_t)stream;
  const size_t n = (size_t)N * K;
  const int nb = pq_stats_blocks(n);
  if (int e = pq_launch_wstats_partial(W, w_dtype, n, (double*)workspace, nb, s)) return e;
  return pq_launch_pack(W, w_dtype, N, K, (const double*)workspace, nb, packed, packed_t, mu_lambda, s);
}

extern "C" int pq_router_topk(const void* X, const void* Wr, int32_t dtype, int32_t T, int32_t K, int32_t E,
                              int32_t k, int32_t* idx, float* gate, float* probs, void* stream) {
  if (int e = check_dtype(dtype)) return e;
  PQ_REQUIRE(T >= 0 && K > 0, PQ_ERR_BAD_ARG, "bad size T=%d K=%d", T, K);
  PQ_REQUIRE(E >= 1 && E <= 64, PQ_ERR_BAD_ARG, "E=%d must be in 1..64", E);
  PQ_REQUIRE(k >= 1 && k <= E, PQ_ERR_BAD_ARG, "k=%d must be in 1..E", k);
  PQ_REQUIRE(K % 8 == 0, PQ_ERR_SHAPE, "K=%d must be a multiple of 8", K);
  if (T == 0) return PQ_OK;
  PQ_REQUIRE(X && Wr && idx && gate, PQ_ERR_BAD_ARG, "NULL buffer");
  PQ_REQUIRE(aligned16(X) && aligned16(Wr), PQ_ERR_SHAPE, "X and Wr must be 16-byte aligned");
  return pq_launch_router(X, Wr, dtype, T, K, E, k, idx, gate, probs, (hipStream_t)stream);
}

extern "C" int pq_onebit_acc(const int8_t* Xq, const uint32_t* packed, int32_t T, int32_t K, int32_t N,
                             int32_t* acc, void* stream) {
  PQ_REQUIRE(T >= 0 && K > 0 && N > 0, PQ_ERR_BAD_ARG, "bad size T=%d K=%d N=%d", T, K, N);
  PQ_REQUIRE(K % 32 == 0, PQ_ERR_SHAPE, "K=%d must be a multiple of 32", K);
  if (T == 0) return PQ_OK;
  PQ_REQUIRE(Xq && packed && acc, PQ_ERR_BAD_ARG, "NULL buffer");
  PQ_REQUIRE(N % 8 == 0 && aligned16(acc), PQ_ERR_SHAPE, "N=%d must be a multiple of 8 and acc 16-byte aligned", N);
  PQ_REQUIRE(aligned16(Xq) && aligned16(packed), PQ_ERR_SHAPE, "Xq and packed must be 16-byte aligned");
  pq_operand A{Xq, K, PQ_SRC_KC8, nullptr};
  pq_operand B{packed, K / 8, PQ_SRC_BITS8, nullptr};
  pq_epilogue e = epi_zero();
  e.C = acc; e.ldc = N; e.out_kind = PQ_OUT_I32;
  return pq_launch_gemm(T, N, K, A, B, e, (hipStream_t)stream);
}

extern "C" size_t pq_linear_ctx_bytes(const pq_linear_desc* d) {
  if (check_desc(d, false) != PQ_OK) return 0;
  return make_layout(*d).ctx_total;
}

extern "C" size_t pq_linear_workspace_bytes(const pq_linear_desc* d) {
  if (check_desc(d, false) != PQ_OK) return 0;
  return make_layout(*d).ws_total;
}

namespace {
struct hp8_layout { size_t Aq, gA, At, Bq, gB, Bt, H, Hq, gH, Ht, ctx_total, dH, splitk, splitk2, splitk_bytes, splitk2_bytes, ws_total; };
hp8_layout make_hp8_layout(int T, int K, int N, int r) {
  hp8_layout L;
  const size_t t = T, k = K, n = N, rr = r;
  cursor c;
  L.Aq = c.take(rr * k); L.gA = c.take(rr * sizeof(float)); L.At = c.take(rr * k * 2);
  L.Bq = c.take(n * rr); L.gB = c.take(n * sizeof(float)); L.Bt = c.take(n * rr * 2);
  L.H = c.take(t * rr * 2); L.Hq = c.take(t * rr); L.gH = c.take(t * sizeof(float)); L.Ht = c.take(t * rr * 2);
  L.ctx_total = c.off;
  cursor w;
  L.dH = w.take(t * rr * 2);
  size_t sk = 0;
  const int shapes[4][3] = {{T, r, N}, {N, r, T}, {r, K, T}, {T, K, r}};
  for (const auto& sh : shapes) {
    if (sh[0] <= 0 || sh[1] <= 0) continue;
    const size_t b = pq_plan_gemm(sh[0], sh[1], sh[2]).ws_bytes;
    if (b > sk) sk = b;
  }
  if (T > 0) {   // the int8 H product splits its contraction (int32 slabs)
    const size_t b = pq_plan_gemm(T, r, K, true, true).ws_bytes;
    if (b > sk) sk = b;
  }
  const pq_pair_plan pair = pq_plan_pair(T, N, r, r, K);
  if (pair.ws0 > sk) sk = pair.ws0;
  L.splitk = w.take(sk);
  L.splitk_bytes = sk;
  const size_t alone = (r > 0 && K > 0) ? pq_plan_gemm(r, K, T).ws_bytes : 0;
  L.splitk2_bytes = pair.ws1 > alone ? pair.ws1 : alone;
  L.splitk2 = w.take(L.splitk2_bytes);   // dA's slabs when dB and dA share a launch
  L.ws_total = w.off;
  return L;
}
}  // namespace
// pq_hp_int8_fwd; rows_done: the rows of A and B are already on their grid in ctx
static int hp_int8_fwd_impl(const int8_t* Xq, const float* gamma_x, const void* A, const void* B, int32_t dtype, int32_t T, int32_t K,
                            int32_t N, int32_t r, float alpha, void* Y, int32_t accumulate, void* ctx, size_t ctx_bytes, void* workspace,
                            size_t workspace_bytes, void* stream, bool rows_done);

// ---------------------------------------------------------------------------------------------
// Forward: [stats -> pack] -> quantise -> int8 MFMA GEMM with de-quantising epilogue -> hp branch
// ---------------------------------------------------------------------------------------------
// prequant: the quantised activations (codes, gamma, q/gamma) are already in ctx, the weight statistics' first stage in
// the workspace, and X is what the high-precision branch reads (the normalising entry point runs the fused quantiser first)
static int linear_fwd_impl(const pq_linear_desc* d, const void* X, const void* W_or_packed,
                           const float* mu_lambda, const void* hpA, const void* hpB, const void* Wr, void* Y,
                           void* ctx, size_t ctx_bytes, void* workspace, size_t workspace_bytes, void* stream, bool prequant) {
  if (int e = check_desc(d, false)) return e;
  const lin_layout L = make_layout(*d);
  const bool routed = d->n_experts > 1 && d->hp_rank > 0;                 // Sec. 3.3: top-k routed low-rank experts
  const bool hp8 = d->hp_kind == PQ_HP_LOWRANK_INT8 && d->hp_rank > 0;    // Sec. 3.2: the branch in its INT8 form
  // r is the rank of the dense 16-bit branch handled inline below; the other two forms run behind the 1-bit GEMM
  const int T = d->tokens, K = d->d_in, N = d->d_out, r = (routed || hp8) ? 0 : d->hp_rank;
  PQ_REQUIRE((d->tokens == 0 || (X && Y)) && W_or_packed && workspace, PQ_ERR_BAD_ARG, "NULL buffer (X, W, Y or workspace)");
  PQ_REQUIRE(d->hp_rank == 0 || (hpA && hpB), PQ_ERR_BAD_ARG, "hp_rank=%d but hpA/hpB is NULL", d->hp_rank);
  PQ_REQUIRE(!routed || Wr, PQ_ERR_BAD_ARG, "n_experts=%d needs the router weights Wr", d->n_experts);
  PQ_REQUIRE(!(routed || hp8) || ctx, PQ_ERR_BAD_ARG, "routed experts and the INT8 high-precision branch need a ctx");
  PQ_REQUIRE(aligned16(Wr), PQ_ERR_SHAPE, "Wr must be 16-byte aligned");
  PQ_REQUIRE(d->w_kind == PQ_W_MASTER || mu_lambda, PQ_ERR_BAD_ARG, "packed weights need mu_lambda");
  PQ_REQUIRE(d->w_kind == PQ_W_PACKED || ctx, PQ_ERR_BAD_ARG, "latent weights need a ctx to hold the packed bits");
  PQ_REQUIRE(aligned16(X) && aligned16(W_or_packed) && aligned16(Y) && aligned16(workspace) && aligned16(ctx) &&
                 aligned16(hpA) && aligned16(hpB), PQ_ERR_SHAPE, "buffers must be 16-byte aligned");
  PQ_REQUIRE(workspace_bytes >= L.ws_base, PQ_ERR_WORKSPACE, "workspace too small: %zu < %zu", workspace_bytes, L.ws_base);
  PQ_REQUIRE(!ctx || ctx_bytes >= L.ctx_total, PQ_ERR_WORKSPACE, "ctx too small: %zu < %zu", ctx_bytes, L.ctx_total);
  hipStream_t s = (hipStream_t)stream;
  char* cx = (char*)ctx;
  char* ws = (char*)workspace;
  const pq_scratch sk_ws{ws + L.splitk, L.splitk_bytes};
  const bool bf16 = d->io_dtype == PQ_BF16;
  const int ok = out_kind_of(d->io_dtype);

  int8_t* Xq = (int8_t*)(ctx ? cx + L.Xq : ws + L.w_Xq);
  float* gamma = (float*)(ctx ? cx + L.gamma : ws + L.w_gamma);
  uint16_t* Xt = (ctx && bf16) ? (uint16_t*)(cx + L.Xt) : nullptr;
  bool quant_done = prequant;
  void* H = r > 0 ? (ctx ? (void*)(cx + L.H) : (void*)(ws + L.w_H)) : nullptr;
  // H = X A^T.  A rank of 128 over many tokens takes the streaming rank-r kernel (whole contraction per workgroup,
  // nothing to reduce); other shapes go through the tile engine, which may split the contraction.
  bool H_skinny = false;
  if (r > 0 && bf16 && T > 0) {
    pq_operand A{X, K, PQ_SRC_KC16, nullptr}, B{hpA, K, PQ_SRC_KC16, nullptr};
    pq_epilogue e = epi_zero();
    e.C = H; e.ldc = r; e.out_kind = ok;
    H_skinny = pq_skinny_applies(T, r, K, A, B, e);
  }
  auto H_ref = [&]() {
    pq_epilogue e = epi_zero();
    e.C = H; e.ldc = r; e.out_kind = PQ_OUT_F32;
    return ref_problem(PQ_REF_CC, T, r, K, {X, K, PQ_SRC_KC32, nullptr}, {hpA, K, PQ_SRC_KC32, nullptr}, e);
  };
  auto launch_H = [&](bool defer) -> int {
    pq_epilogue e = epi_zero();
    e.C = H; e.ldc = r; e.out_kind = ok; e.defer_reduce = defer ? 1 : 0;
    if (!bf16) {
      pq_ref_problem p = H_ref();
      return pq_launch_ref(&p, 1, nullptr, 0, s, PQP_GEMM_HP_H);
    }
    pq_operand A{X, K, PQ_SRC_KC16, nullptr};
    pq_operand B{hpA, K, PQ_SRC_KC16, nullptr};
    if (H_skinny) return pq_launch_skinny(T, K, A, B, e, s, PQP_GEMM_HP_H);
    return pq_launch_gemm(T, r, K, A, B, e, s, PQP_GEMM_HP_H, sk_ws);
  };
  // The weight statistics' first stage and the activation quantiser share a launch (rows of up to 8192 elements stay
  // in registers); when H = X A^T splits its contraction it goes first and the sum of its slabs rides along too.
  // Packed weights have no statistics to take: the quantiser and the slabs' sum share the launch there.
  const int H_splits = bf16 && r > 0 && T > 0 ? (H_skinny ? 1 : pq_plan_gemm(T, r, K).splits) : 0;
  const bool combo = !prequant && T > 0 && K <= (bf16 ? 8192 : 4096) && (d->w_kind == PQ_W_MASTER || H_splits > 1);
  bool H_done = false;
  if (combo && bf16 && r > 0) {
    if (int e = launch_H(H_splits > 1)) return e;
    H_done = true;
  }
  // routed experts: the router (with the statistics and the quantiser where they take it), and what orders its slots
  pq_router_job route;
  pq_place place;
  memset(&route, 0, sizeof(route));
  memset(&place, 0, sizeof(place));
  bool routed_done = false;
  if (routed) {
    const int E = d->n_experts, rt = pq_router_tokens(E);
    route = pq_router_job{Wr, E, d->top_k, (int*)(cx + L.idx), (float*)(cx + L.gate), (float*)(cx + L.probs), (int*)(ws + L.hist)};
    place = pq_place{route.hist, (T + rt - 1) / rt, rt, T, d->top_k, E, K, route.idx, (int*)(cx + L.counts), (int*)(cx + L.offsets), (int*)(cx + L.perm),
                     (int*)(cx + L.inv), (const uint16_t*)X, (uint16_t*)(cx + L.Xp), nullptr, nullptr, nullptr, nullptr};
  }
  auto launch_combo = [&](const void* w, size_t n, double* part, int nb) -> int {
    if (routed && pq_wstats_quant_router_applies(d->n_experts, K, nb + (T + 3) / 4)) {
      quant_done = routed_done = true;
      return pq_launch_wstats_quant_router(w, n, part, nb, X, T, K, Xq, gamma, Xt, route, s);
    }
    const bool sum = H_done && H_splits > 1;
    quant_done = true;
    return pq_launch_wstats_quant(w, d->io_dtype, n, part, nb, X, T, K, Xq, gamma, Xt, s, sum ? (const float*)sk_ws.p : nullptr, H_splits, T, r, H, r);
  };
  const uint32_t* P;
  const float* mulam;
  if (d->w_kind == PQ_W_MASTER) {
    const size_t n = (size_t)N * K;
    const int nb = pq_stats_blocks(n);
    double* part = (double*)(ws + L.stat_partials);
    if (combo) {
      if (int e = launch_combo(W_or_packed, n, part, nb)) return e;
    } else if (!prequant) {
      if (int e = pq_launch_wstats_partial(W_or_packed, d->io_dtype, n, part, nb, s)) return e;
    }
    uint32_t* Pt = (N % 32 == 0) ? (uint32_t*)(cx + L.Pt) : nullptr;
    if (routed && !routed_done)
      if (int e = pq_launch_router(X, Wr, PQ_BF16, T, K, route.E, route.k, route.idx, route.gate, route.probs, s, route.hist)) return e;
    if (routed) {   // the slots' order rides along (with no tokens: empty expert segments for a backward)
      if (int e = pq_launch_pack_place(W_or_packed, N, K, part, nb, (uint32_t*)(cx + L.P), Pt, (float*)(cx + L.mulam), place, s)) return e;
    } else if (hp8) {   // the rows of A and B on the AbsMax grid ride along
      const hp8_layout H8 = make_hp8_layout(T, K, N, d->hp_rank);
      char* c8 = cx + L.hp8;
      const pq_quant_rows_job jobs[2] = {{hpA, d->hp_rank, K, (int8_t*)(c8 + H8.Aq), (float*)(c8 + H8.gA), (uint16_t*)(c8 + H8.At)},
                                         {hpB, N, d->hp_rank, (int8_t*)(c8 + H8.Bq), (float*)(c8 + H8.gB), (uint16_t*)(c8 + H8.Bt)}};
      if (int e = pq_launch_pack_quant_rows(W_or_packed, N, K, part, nb, (uint32_t*)(cx + L.P), Pt, (float*)(cx + L.mulam), jobs, s)) return e;
    } else if (!bf16 && r > 0 && pq_ref_rides(T, r, K)) {   // H needs nothing of the weight: a launch less
      if (int e = pq_launch_ref_pack(H_ref(), (const float*)W_or_packed, N, K, part, nb, (uint32_t*)(cx + L.P), Pt, (float*)(cx + L.mulam), s)) return e;
      H_done = true;
    } else if (int e = pq_launch_pack(W_or_packed, d->io_dtype, N, K, part, nb, (uint32_t*)(cx + L.P), Pt,
                                      (float*)(cx + L.mulam), s)) return e;
    P = (const uint32_t*)(cx + L.P);
    mulam = (const float*)(cx + L.mulam);
  } else {
    P = (const uint32_t*)W_or_packed;
    mulam = mu_lambda;
    if (combo)
      if (int e = launch_combo(nullptr, 0, nullptr, 0)) return e;
    if (routed) {
      if (int e = pq_launch_router(X, Wr, PQ_BF16, T, K, route.E, route.k, route.idx, route.gate, route.probs, s, route.hist)) return e;
      if (int e = pq_launch_pack_place(nullptr, N, K, nullptr, 0, nullptr, nullptr, nullptr, place, s)) return e;
    }
  }
  if (T == 0) return PQ_OK;   // the weight side is prepared, so a backward with no tokens is well defined

  if (!quant_done)
    if (int e = pq_launch_quant_act(X, d->io_dtype, T, K, Xq, gamma, Xt, s)) return e;

  // bf16 I/O with a live hp branch: the rank-r product H B^T is accumulated into the 1-bit GEMM's tile
  // (the fused form carries beta / alpha through the tile: only while that ratio stays far from the fp32 range, otherwise
  // the two branches are scaled separately as in the Sec. 3.2 sum)
  const bool fuse_hp = bf16 && r > 0 && d->alpha != 0.0f && fabsf(d->alpha) >= 9.5367431640625e-7f * fabsf(d->beta) &&
                       pq_plan_fuses(pq_plan_gemm(T, N, K, true, true, PQ_PLAN_SIGNS));
  if (r > 0 && !H_done)
    if (int err = launch_H(false)) return err;
  if (!bf16 && r > 0 && d->alpha != 0.0f && pq_ref_linear_applies(T, N, K))   // both branches in one launch
    return pq_launch_ref_linear({Xq, P, mulam + 1, gamma, {H, r, PQ_SRC_KC32, nullptr}, {hpB, r, PQ_SRC_KC32, nullptr}, (float*)Y, T, N, K, r,
                                 d->alpha, d->beta}, s);
  {  // 1-bit branch: Y = fl32(fl32(beta*lambda)/gamma_t) * acc   [+ alpha * H B^T when fused]
    pq_operand A{Xq, K, PQ_SRC_KC8, nullptr};
    pq_operand B{P, K / 8, PQ_SRC_BITS8, nullptr};
    pq_epilogue e = epi_zero();
    e.C = Y; e.ldc = N; e.out_kind = ok; e.split_int8 = bf16 ? 1 : 0;
    if (fuse_hp) {   // Y = alpha * ( (beta*lambda/alpha/gamma_t) * acc + H B^T )
      pq_phase2 p2;
      p2.A2 = pq_operand{H, r, PQ_SRC_KC16, nullptr};
      p2.B2 = pq_operand{hpB, r, PQ_SRC_KC16, nullptr};
      p2.K2 = r; p2.scale1 = d->beta / d->alpha; p2.dev_scale1 = mulam + 1; p2.row_div1 = gamma;
      e.scale = d->alpha;
      if (int err = pq_launch_gemm(T, N, K, A, B, e, s, PQP_GEMM_ONEBIT, sk_ws, nullptr, &p2)) return err;
    } else {
      e.scale = d->beta; e.dev_scale = mulam + 1; e.row_div = gamma;
      if (int err = pq_launch_gemm(T, N, K, A, B, e, s, PQP_GEMM_ONEBIT, sk_ws)) return err;
    }
  }
  if (r > 0 && !fuse_hp && d->alpha != 0.0f) {  // Y += alpha * H B^T
    pq_epilogue e = epi_zero();
    e.C = Y; e.ldc = N; e.out_kind = ok; e.accumulate = 1; e.scale = d->alpha;
    if (bf16) {
      pq_operand A{H, r, PQ_SRC_KC16, nullptr};
      pq_operand B{hpB, r, PQ_SRC_KC16, nullptr};
      if (int err = pq_launch_gemm(T, N, r, A, B, e, s, PQP_GEMM_HP_Y, sk_ws)) return err;
    } else {
      pq_ref_problem p = ref_problem(PQ_REF_CC, T, N, r, {H, r, PQ_SRC_KC32, nullptr}, {hpB, r, PQ_SRC_KC32, nullptr}, e);
      if (int err = pq_launch_ref(&p, 1, nullptr, 0, s, PQP_GEMM_HP_Y)) return err;
    }
  }
  if (hp8)   // Y += alpha * B~ Q(A~ Q(x)) on the codes and gamma formed above
    return hp_int8_fwd_impl(Xq, gamma, hpA, hpB, PQ_BF16, T, K, N, d->hp_rank, d->alpha, Y, 1, cx + L.hp8, L.hp8_bytes,
                            ws + L.hp8_ws, L.hp8_ws_bytes, stream, d->w_kind == PQ_W_MASTER);
  if (routed) {
    // slots in expert order (above) -> H_e = X_e A_e^T -> Y_e = H_e B_e^T -> gate-weighted combine
    const int E = d->n_experts, k = d->top_k, S = T * k, re = d->hp_rank;
    pq_gemm_group g1{place.offsets, E, 1, 0, 0, S};
    {
      pq_operand A{cx + L.Xp, K, PQ_SRC_KC16, nullptr};
      pq_operand B{hpA, K, PQ_SRC_KC16, nullptr};
      pq_epilogue e = epi_zero();
      e.C = cx + L.Hs; e.ldc = re; e.out_kind = PQ_OUT_BF16;
      g1.b_stride = (long)re * K;
      if (int err = pq_launch_gemm(S, re, K, A, B, e, s, PQP_GEMM_EXPERT, sk_ws, &g1)) return err;
    }
    {
      pq_operand A{cx + L.Hs, re, PQ_SRC_KC16, nullptr};
      pq_operand B{hpB, re, PQ_SRC_KC16, nullptr};
      pq_epilogue e = epi_zero();
      e.C = cx + L.Ys; e.ldc = N; e.out_kind = PQ_OUT_BF16;
      g1.b_stride = (long)N * re;
      if (int err = pq_launch_gemm(S, N, re, A, B, e, s, PQP_GEMM_EXPERT, sk_ws, &g1)) return err;
    }
    return pq_launch_combine_fwd(Y, cx + L.Ys, place.inv, route.gate, d->alpha, T, k, N, s);
  }
  return PQ_OK;
}

extern "C" int pq_linear_fwd(const pq_linear_desc* d, const void* X, const void* W_or_packed,
                             const float* mu_lambda, const void* hpA, const void* hpB, const void* Wr, void* Y,
                             void* ctx, size_t ctx_bytes, void* workspace, size_t workspace_bytes, void* stream) {
  return linear_fwd_impl(d, X, W_or_packed, mu_lambda, hpA, hpB, Wr, Y, ctx, ctx_bytes, workspace, workspace_bytes, stream, false);
}

// ---------------------------------------------------------------------------------------------
// STE backward
// ---------------------------------------------------------------------------------------------
// The two halves of pq_hp_int8_bwd that do not touch dX, on checked arguments.  dH = alpha dY B~, with the per-workgroup partial
// sums of <dY, Y_hp> (= d alpha) left in red_a when it is not NULL; then dB and dA, two scalar reductions (may be NULL) riding
// along where the launch has room for them.
static int hp_int8_dh(const void* dY, int T, int N, int r, float alpha, const char* cx, const hp8_layout& L, char* ws, double* red_a, hipStream_t s);
static int hp_int8_factor_grads(const void* dY, const void* Xt, int T, int K, int N, int r, float alpha, const char* cx, const hp8_layout& L,
                                float* dA, float* dB, char* ws, const pq_reduce_job* jobs, bool* jobs_done, hipStream_t s,
                                const pq_grads* along);

// fp32 I/O: the same products at reference precision; large ones of dX and dW as exact integer products of fixed-point digits
// (pq_fixed.hip), whose sums the launches below finish.  What depends on nothing (dW, dH, dB) is one launch, what needs dH
// (dX with dH A in the same sums, dA) and the two scalar reductions a second one: six products and a reduction in a row
// left most of the chip idle at every size, and at 64 tokens their starts were most of the time.
// fx: the region of the digits and their sums, or NULL for the fp64 products alone.
static int linear_bwd_f32(const pq_linear_desc* d, const lin_layout& L, const void* dY, const void* X, const void* W, const void* hpA,
                          const void* hpB, const char* cx, void* dX, float* dW, float* dhpA, float* dhpB, float* dalpha_dbeta, char* ws, char* fx,
                          hipStream_t s) {
  const int T = d->tokens, K = d->d_in, N = d->d_out, r = d->hp_rank;
  const float* mulam = (const float*)(cx + L.mulam);
  double* red_a = (double*)(ws + L.red_a);
  double* red_b = (double*)(fx ? fx + L.fx_red_b : ws + L.red_b);
  const void* H = cx + L.H;
  void* dH = ws + L.dH;
  pq_ref_problem p[PQ_REF_MAX];
  int n = 0;
  double *SW = fx ? (double*)(fx + L.fx_SW) : nullptr, *SX = fx ? (double*)(fx + L.fx_SX) : nullptr;
  if (fx) {                          // dY S and (dY / gamma)^T q from the digits of dY's rows and columns
    int8_t *drow = (int8_t*)(fx + L.fx_drow), *dcol = (int8_t*)(fx + L.fx_dcol), *qT = (int8_t*)(fx + L.fx_qT), *signs = (int8_t*)(fx + L.fx_signs);
    int *rexp = (int*)(fx + L.fx_rexp), *cexp = (int*)(fx + L.fx_cexp);
    if (int err = pq_launch_fixed_split((const float*)dY, (const float*)(cx + L.gamma), (const int8_t*)(cx + L.Xq), T, N, K, drow, rexp, dcol, cexp, qT,
                                        (uint32_t*)(fx + L.fx_colmax), (int*)(fx + L.fx_counts), (const uint32_t*)(cx + L.Pt), signs, s)) return err;
    if (int err = pq_launch_fixed_products(drow, rexp, signs, SX, dcol, cexp, qT, SW, T, N, K, s)) return err;
  }
  auto add_dW = [&] {  // dW = beta * dY^T (q / gamma)  [masked];  d beta = lambda * sum S .* (dY^T (q / gamma))
    pq_epilogue e = epi_zero();
    e.C = dW; e.ldc = K; e.scale = d->beta;
    e.sign_bytes = (const uint8_t*)(cx + L.P); e.ld_sign = K / 8; e.partials = red_b;
    if (d->ste_mode == PQ_STE_CLIP) { e.maskW = W; e.mu_dev = mulam; e.tau = d->ste_tau; }
    p[n] = ref_problem(fx ? PQ_REF_SUM_SS8 : PQ_REF_SS8, N, K, T, {dY, N, PQ_SRC_KS32, nullptr},
                       {cx + L.Xq, K, PQ_SRC_KS8, (const float*)(cx + L.gamma)}, e);
    p[n].sums = SW; p[n].exps = fx ? (const int*)(fx + L.fx_cexp) : nullptr;
    p[n].counts = fx ? (const int*)(fx + L.fx_counts) : nullptr;
    ++n;
  };
  if (!fx) add_dW();                 // (the longest first: products before sums of digits)
  if (r > 0) {
    pq_epilogue e = epi_zero();      // dB = alpha * dY^T H
    e.C = dhpB; e.ldc = r; e.scale = d->alpha;
    p[n++] = ref_problem(PQ_REF_SS, N, r, T, {dY, N, PQ_SRC_KS32, nullptr}, {H, r, PQ_SRC_KS32, nullptr}, e);
    e = epi_zero();                  // dH = alpha * dY B ; d alpha = <H, dY B>
    e.C = dH; e.ldc = r; e.scale = d->alpha; e.dot_comp = H; e.ld_comp = r; e.partials = red_a;
    p[n++] = ref_problem(PQ_REF_CS, T, r, N, {dY, N, PQ_SRC_KC32, nullptr}, {hpB, r, PQ_SRC_KS32, nullptr}, e);
  }
  if (fx) add_dW();
  if (int err = pq_launch_ref(p, n, nullptr, 0, s, PQP_GEMM_DW)) return err;
  const pq_reduce_job jobs[2] = {{red_a, (T > 0 && r > 0) ? pq_ref_red_blocks(T, r, N) : 0, 1.0f, nullptr, dalpha_dbeta},
                                 {red_b, fx ? pq_ref_red_blocks(N, K, -1) : L.n_red_b, 1.0f, mulam + 1, dalpha_dbeta + 1}};
  n = 0;
  auto add_dX = [&] {                // dX = beta * lambda * dY S + dH A
    pq_epilogue e = epi_zero();
    e.C = dX; e.ldc = K;
    p[n] = ref_problem(fx ? PQ_REF_SUM_CBITS : PQ_REF_CBITS, T, K, N, {dY, N, PQ_SRC_KC32, nullptr}, {cx + L.Pt, N / 8, PQ_SRC_BITSF, nullptr}, e);
    p[n].sums = SX; p[n].exps = fx ? (const int*)(fx + L.fx_rexp) : nullptr;
    p[n].scale1 = d->beta; p[n].dev_scale1 = mulam + 1;
    if (r > 0) { p[n].K2 = r; p[n].A2 = pq_operand{dH, r, PQ_SRC_KC32, nullptr}; p[n].B2 = pq_operand{hpA, K, PQ_SRC_KS32, nullptr}; }
    ++n;
  };
  if (!fx) add_dX();
  if (r > 0) {                       // dA = dH^T X   (dH already carries alpha)
    pq_epilogue e = epi_zero();
    e.C = dhpA; e.ldc = K;
    p[n++] = ref_problem(PQ_REF_SS, r, K, T, {dH, r, PQ_SRC_KS32, nullptr}, {X, K, PQ_SRC_KS32, nullptr}, e);
  }
  if (fx) add_dX();
  return pq_launch_ref(p, n, jobs, 2, s, PQP_GEMM_DX);
}

// fx_at: where the region of fp32 digits lies when it does not follow ws_base in the workspace.
static int linear_bwd_impl(const pq_linear_desc* d, const void* dY, const void* X, const void* W,
                           const void* hpA, const void* hpB, const void* Wr, const void* ctx, size_t ctx_bytes,
                           void* dX, float* dW, float* dhpA, float* dhpB, float* dWr, float* dalpha_dbeta,
                           void* workspace, size_t workspace_bytes, void* stream, char* fx_at) {
  if (int e = check_desc(d, true)) return e;
  const lin_layout L = make_layout(*d);
  const bool routed = d->n_experts > 1 && d->hp_rank > 0;
  const bool hp8 = d->hp_kind == PQ_HP_LOWRANK_INT8 && d->hp_rank > 0;
  const int T = d->tokens, K = d->d_in, N = d->d_out, r = (routed || hp8) ? 0 : d->hp_rank;
  PQ_REQUIRE((d->tokens == 0 || (dY && X && dX)) && ctx && dW && dalpha_dbeta && workspace, PQ_ERR_BAD_ARG, "NULL buffer");
  PQ_REQUIRE(d->hp_rank == 0 || (hpA && hpB && dhpA && dhpB), PQ_ERR_BAD_ARG, "hp_rank=%d but an hp buffer is NULL", d->hp_rank);
  PQ_REQUIRE(!routed || (Wr && dWr), PQ_ERR_BAD_ARG, "n_experts=%d needs Wr and dWr", d->n_experts);
  PQ_REQUIRE(aligned16(Wr) && aligned16(dhpA) && aligned16(dhpB), PQ_ERR_SHAPE, "buffers must be 16-byte aligned");
  PQ_REQUIRE(d->ste_mode == PQ_STE_IDENTITY || W, PQ_ERR_BAD_ARG, "PQ_STE_CLIP needs the latent W");
  PQ_REQUIRE(aligned16(dY) && aligned16(X) && aligned16(ctx) && aligned16(dX) && aligned16(dW) && aligned16(workspace) &&
                 aligned16(hpA) && aligned16(hpB) && aligned16(W), PQ_ERR_SHAPE, "buffers must be 16-byte aligned");
  PQ_REQUIRE(workspace_bytes >= L.ws_base, PQ_ERR_WORKSPACE, "workspace too small: %zu < %zu", workspace_bytes, L.ws_base);
  PQ_REQUIRE(ctx_bytes >= L.ctx_total, PQ_ERR_WORKSPACE, "ctx too small: %zu < %zu", ctx_bytes, L.ctx_total);
  hipStream_t s = (hipStream_t)stream;
  const char* cx = (const char*)ctx;
  char* ws = (char*)workspace;
  const pq_scratch sk_ws{ws + L.splitk, L.splitk_bytes};
  const bool bf16 = d->io_dtype == PQ_BF16;
  const int ok = out_kind_of(d->io_dtype);
  const float* mulam = (const float*)(cx + L.mulam);
  const void* H = cx + L.H;
  void* dH = ws + L.dH;
  double* red_a = (double*)(ws + L.red_a);
  double* red_b = (double*)(ws + L.red_b);
  if (!bf16) {
    char* fx = L.fx_bytes == 0 ? nullptr : fx_at ? fx_at : workspace_bytes >= L.ws_total ? ws + L.ws_base : nullptr;
    return linear_bwd_f32(d, L, dY, X, W, hpA, hpB, cx, dX, dW, dhpA, dhpB, dalpha_dbeta, ws, fx, s);
  }
  int n_red_a = r > 0 ? pq_plan_gemm(T, r, N).red_blocks : 0;   // partial sums of d alpha that the dH GEMM leaves

  if (T > 0 && r > 0) {  // dH = alpha * dY B ; d alpha = <H, dY B>
    pq_operand A{dY, N, PQ_SRC_KC16, nullptr};
    pq_operand B{hpB, r, PQ_SRC_KS16, nullptr};
    pq_epilogue e = epi_zero();
    e.C = dH; e.ldc = r; e.out_kind = ok; e.scale = d->alpha;
    e.dot_comp = H; e.ld_comp = r; e.comp_kind = ok; e.partials = red_a;
    if (pq_skinny_applies(T, r, N, A, B, e)) {   // many tokens at rank 128: nothing to split or reduce
      n_red_a = pq_skinny_blocks(T);
      if (int err = pq_launch_skinny(T, N, A, B, e, s, PQP_GEMM_DH)) return err;
    } else if (int err = pq_launch_gemm(T, r, N, A, B, e, s, PQP_GEMM_DH, sk_ws)) return err;
  }

  // INT8 branch: STE on the de-quantised factors; its dH GEMM leaves the partials of d alpha
  hp8_layout H8;
  memset(&H8, 0, sizeof(H8));
  if (hp8) H8 = make_hp8_layout(T, K, N, d->hp_rank);
  if (hp8 && T > 0) {
    n_red_a = pq_plan_gemm(T, d->hp_rank, N).red_blocks;
    if (int e = hp_int8_dh(dY, T, N, d->hp_rank, d->alpha, cx + L.hp8, H8, ws + L.hp8_ws, red_a, s)) return e;
  }
  pq_gemm_call set[2];
  int n_set = 1;
  pq_grads grads;                                    // what is left to the launch of the factor gradients
  grads.has_x = false;
  grads.sk = sk_ws;
  const bool dW_last = T > 0 && (hp8 || r > 0);
  if (T > 0) {  // dX = beta*lambda * dY S  (+ dH A, fused into the same tile)
    pq_operand A{dY, N, PQ_SRC_KC16, nullptr};
    pq_operand B{cx + L.Pt, N / 8, PQ_SRC_BITS16, nullptr};
    pq_epilogue e = epi_zero();
    e.C = dX; e.ldc = K; e.out_kind = ok;
    // the branch's share of dX: dH A, with the INT8 form on its de-quantised rows
    const int r2 = hp8 ? d->hp_rank : r;
    const void* dH2 = hp8 ? (const void*)(ws + L.hp8_ws + H8.dH) : dH;
    const void* A2p = hp8 ? (const void*)(cx + L.hp8 + H8.At) : hpA;
    const bool fuse = r2 > 0 && pq_plan_fuses(pq_plan_gemm(T, K, N, false, false, PQ_PLAN_SIGNS));
    if (fuse) {
      pq_phase2& p2 = grads.p2;
      p2.A2 = pq_operand{dH2, r2, PQ_SRC_KC16, nullptr};
      p2.B2 = pq_operand{A2p, K, PQ_SRC_KS16, nullptr};
      p2.K2 = r2; p2.scale1 = d->beta; p2.dev_scale1 = mulam + 1; p2.row_div1 = nullptr;
      grads.x = pq_gemm_call{T, K, N, A, B, e, nullptr, PQP_GEMM_DX};
      grads.has_x = true;
    } else {
      e.scale = d->beta; e.dev_scale = mulam + 1;
      if (r2 == 0) {                 // nothing between it and dW: they go together
        set[1] = pq_gemm_call{T, K, N, A, B, e, nullptr, PQP_GEMM_DX};
        n_set = 2;
      } else if (int err = pq_launch_gemm(T, K, N, A, B, e, s, PQP_GEMM_DX, sk_ws)) return err;
      if (r2 > 0) {
        pq_operand A2{dH2, r2, PQ_SRC_KC16, nullptr};
        pq_operand B2{A2p, K, PQ_SRC_KS16, nullptr};
        pq_epilogue e2 = epi_zero();
        e2.C = dX; e2.ldc = K; e2.out_kind = ok; e2.accumulate = 1;
        // (the INT8 branch's products split into the branch's own section, which is sized for them)
        const pq_scratch sk2 = hp8 ? pq_scratch{ws + L.hp8_ws + H8.splitk, H8.splitk_bytes} : sk_ws;
        if (int err = pq_launch_gemm(T, K, r2, A2, B2, e2, s, PQP_GEMM_DX_HP, sk2)) return err;
      }
    }
  }
  {  // dW = beta * (dY/gamma)^T q  [masked];  d beta = lambda * sum S .* (dY/gamma)^T q
    pq_operand A{dY, N, PQ_SRC_KS16, nullptr};
    pq_operand B{cx + L.Xt, K, PQ_SRC_KS16, nullptr};
    pq_epilogue e = epi_zero();
    e.C = dW; e.ldc = K; e.out_kind = PQ_OUT_F32; e.scale = d->beta;
    e.sign_bytes = (const uint8_t*)(cx + L.P); e.ld_sign = K / 8; e.partials = red_b;
    if (d->ste_mode == PQ_STE_CLIP) {
      e.maskW = W; e.mask_kind = ok; e.mu_dev = mulam; e.tau = d->ste_tau;
    }
    set[0] = pq_gemm_call{N, K, T, A, B, e, nullptr, PQP_GEMM_DW};
    grads.w = set[0];
    if (dW_last) {                   // with the factor gradients below
    } else if (n_set == 2) {
      if (int err = pq_launch_gemm_set(set, 2, s, sk_ws)) return err;
    } else if (int err = pq_launch_gemm(N, K, T, A, B, e, s, PQP_GEMM_DW, sk_ws)) return err;
  }
  if (routed) {
    // Sec. 3.3 backward: upstream of expert e's output for slot (t, j) is alpha gate_tj dY_t; the gate itself
    // receives dgate_tj = alpha <dY_t, Y_e(x_t)> and is differentiated through the softmax into Wr and X.
    const int E = d->n_experts, k = d->top_k, S = T * k, re = d->hp_rank;
    const int* idx = (const int*)(cx + L.idx);
    const float* gate = (const float*)(cx + L.gate);
    const int* offsets = (const int*)(cx + L.offsets);
    const int* perm = (const int*)(cx + L.perm);
    const int* inv = (const int*)(cx + L.inv);
    float* rd = (float*)(ws + L.rd);
    n_red_a = S > 0 ? pq_rowdot_blocks(S) : 0;
    // row dots with the experts' outputs, and dYp = alpha gate dY in slot order
    if (int e = pq_launch_slot_grad(dY, cx + L.Ys, perm, gate, d->alpha, true, k, S, N, ws + L.dYp, rd, red_a, s)) return e;
    pq_gemm_group g1{offsets, E, 1, 0, 0, S};
    pq_gemm_group g2{offsets, E, 2, 0, 0, S};
    if (S > 0) {  // dH_e = (alpha gate dY)_e B_e
      pq_operand A{ws + L.dYp, N, PQ_SRC_KC16, nullptr};
      pq_operand B{hpB, re, PQ_SRC_KS16, nullptr};
      pq_epilogue e = epi_zero();
      e.C = ws + L.dHs; e.ldc = re; e.out_kind = PQ_OUT_BF16;
      g1.b_stride = (long)N * re;
      if (int err = pq_launch_gemm(S, re, N, A, B, e, s, PQP_GEMM_EXPERT, sk_ws, &g1)) return err;
    }
    // per-expert weight gradients (the contraction runs over the expert's slots), and dXs = dH_e A_e in slot order, which the
    // combination scatters back with the router's share
    pq_gemm_call c[3];
    pq_gemm_group gB = g2, gA = g2;
    {
      pq_epilogue e = epi_zero();
      e.C = dhpB; e.ldc = re; e.out_kind = PQ_OUT_F32;
      gB.c_stride = (long)N * re;
      c[0] = pq_gemm_call{N, re, S, {ws + L.dYp, N, PQ_SRC_KS16, nullptr}, {cx + L.Hs, re, PQ_SRC_KS16, nullptr}, e, &gB, PQP_GEMM_EXPERT};
      e.C = dhpA; e.ldc = K;
      gA.c_stride = (long)re * K;
      c[1] = pq_gemm_call{re, K, S, {ws + L.dHs, re, PQ_SRC_KS16, nullptr}, {cx + L.Xp, K, PQ_SRC_KS16, nullptr}, e, &gA, PQP_GEMM_EXPERT};
      e.C = ws + L.dXs; e.out_kind = PQ_OUT_BF16;
      g1.b_stride = (long)re * K;
      c[2] = pq_gemm_call{S, K, re, {ws + L.dHs, re, PQ_SRC_KC16, nullptr}, {hpA, K, PQ_SRC_KS16, nullptr}, e, &g1, PQP_GEMM_EXPERT};
    }
    if (int err = pq_launch_gemm_set(c, 3, s, sk_ws)) return err;
    float* dlogit = (float*)(ws + L.dlogit);
    const pq_reduce_job rj[2] = {{red_a, n_red_a, 1.0f, nullptr, dalpha_dbeta}, {red_b, L.n_red_b, 1.0f, mulam + 1, dalpha_dbeta + 1}};
    if (int e = pq_launch_dwr(rd, inv, idx, (const float*)(cx + L.probs), d->alpha, k, dlogit, X, T, K, E, (float*)(ws + L.dwr), dWr, rj, s)) return e;
    if (int e = pq_launch_combine_bwd(dX, ws + L.dXs, inv, dlogit, Wr, T, k, K, E, s)) return e;
  }
  // d alpha and d beta: both fixed-order sums of per-workgroup partials
  const pq_reduce_job jobs[2] = {{red_a, (T > 0 && (r > 0 || routed || hp8)) ? n_red_a : 0, 1.0f, nullptr, dalpha_dbeta},
                                 {red_b, L.n_red_b, 1.0f, mulam + 1, dalpha_dbeta + 1}};
  bool jobs_done = routed;   // (the routed path's own last reduction carries them)
  if (hp8)
    if (int e = hp_int8_factor_grads(dY, cx + L.Xt, T, K, N, d->hp_rank, d->alpha, cx + L.hp8, H8, dhpA, dhpB, ws + L.hp8_ws, jobs, &jobs_done, s,
                                     dW_last ? &grads : nullptr)) return e;
  if (r > 0 && T > 0) {
    // dB = alpha * dY^T H and dA = dH^T X (dH already carries alpha): two narrow GEMMs over the same contraction,
    // one launch when their plans agree; the two scalar reductions then ride along with their split reduction
    pq_operand A0{dY, N, PQ_SRC_KS16, nullptr}, B0{H, r, PQ_SRC_KS16, nullptr};
    pq_operand A1{dH, r, PQ_SRC_KS16, nullptr}, B1{X, K, PQ_SRC_KS16, nullptr};
    if (int err = pq_launch_gemm_pair_ks16(T, N, r, A0, B0, dhpB, r, d->alpha, r, K, A1, B1, dhpA, K, 1.0f, s, PQP_GEMM_DB, PQP_GEMM_DA,
                                           sk_ws, {ws + L.splitk2, L.splitk2_bytes}, jobs, &jobs_done, &grads)) return err;
  }
  if (!jobs_done)
    if (int err = pq_launch_reduce_partials2(jobs[0].partials, jobs[0].n, 1.0f, nullptr, jobs[0].out, jobs[1].partials, jobs[1].n, 1.0f,
                                             jobs[1].dev_factor, jobs[1].out, s)) return err;
  if (r > 0 && T == 0) {   // no tokens: the factor gradients are the zeros an empty contraction leaves
    pq_operand A{dY, N, PQ_SRC_KS16, nullptr}, B{H, r, PQ_SRC_KS16, nullptr};
    pq_epilogue e = epi_zero();
    e.C = dhpB; e.ldc = r; e.out_kind = PQ_OUT_F32; e.scale = d->alpha;
    if (int err = pq_launch_gemm(N, r, T, A, B, e, s, PQP_GEMM_DB, sk_ws)) return err;
    pq_operand A1{dH, r, PQ_SRC_KS16, nullptr}, B1{X, K, PQ_SRC_KS16, nullptr};
    e.C = dhpA; e.ldc = K; e.scale = 1.0f;
    if (int err = pq_launch_gemm(r, K, T, A1, B1, e, s, PQP_GEMM_DA, sk_ws)) return err;
  }
  return PQ_OK;
}

extern "C" int pq_linear_bwd(const pq_linear_desc* d, const void* dY, const void* X, const void* W,
                             const void* hpA, const void* hpB, const void* Wr, const void* ctx, size_t ctx_bytes,
                             void* dX, float* dW, float* dhpA, float* dhpB, float* dWr, float* dalpha_dbeta,
                             void* workspace, size_t workspace_bytes, void* stream) {
  return linear_bwd_impl(d, dY, X, W, hpA, hpB, Wr, ctx, ctx_bytes, dX, dW, dhpA, dhpB, dWr, dalpha_dbeta, workspace, workspace_bytes, stream, nullptr);
}

// ---------------------------------------------------------------------------------------------
// The linear with its normalisation (Sec. 3.1: Y = (lambda/gamma) W Q(Norm(X))): the fused normalising
// quantiser writes codes, gamma and q/gamma straight into the linear's ctx, the high-precision branch reads
// the stored normalised activations, and the backward chains the linear's dX into the normalisation backward.
// ctx = [linear ctx][x_hat T*K][rstd T]; workspace = [linear workspace][d x_hat T*K][dgain partial rows][fp32 digits].
// ---------------------------------------------------------------------------------------------
namespace {
struct norm_layout { size_t Xn, rstd, ctx_total, dXn, part, ws_base, ws_total; };
norm_layout make_norm_layout(const pq_linear_desc& d, const lin_layout& L) {
  norm_layout n;
  const size_t T = d.tokens, K = d.d_in, es = esize(d.io_dtype);
  cursor c; c.off = pq_align_up(L.ctx_total, 256);
  n.Xn = c.take(T * K * es);
  n.rstd = c.take(T * sizeof(float));
  n.ctx_total = c.off;
  cursor w; w.off = L.ws_base;
  n.dXn = w.take(T * K * es);
  n.part = w.take(pq_rmsnorm_bwd_scratch_bytes(d.tokens, d.d_in) + 256);
  n.ws_base = w.off;
  n.ws_total = w.off + L.fx_bytes;
  return n;
}
int check_norm(const pq_linear_desc* d, bool bwd) {
  const int lim = d->io_dtype == PQ_F32 ? (bwd ? 2048 : 4096) : (bwd ? 4096 : 8192);
  PQ_REQUIRE(d->d_in <= lim, PQ_ERR_SHAPE, "d_in=%d exceeds the row length the fused normalisation keeps in registers (%d)", d->d_in, lim);
  return PQ_OK;
}
}  // namespace

extern "C" size_t pq_linear_norm_ctx_bytes(const pq_linear_desc* d) {
  if (check_desc(d, false) != PQ_OK) return 0;
  return make_norm_layout(*d, make_layout(*d)).ctx_total;
}
extern "C" size_t pq_linear_norm_workspace_bytes(const pq_linear_desc* d) {
  if (check_desc(d, false) != PQ_OK) return 0;
  return make_norm_layout(*d, make_layout(*d)).ws_total;
}

extern "C" int pq_linear_norm_fwd(const pq_linear_desc* d, const void* X, const void* gain, float eps, const void* W,
                                  const void* hpA, const void* hpB, const void* Wr, void* Y, void* ctx, size_t ctx_bytes,
                                  void* workspace, size_t workspace_bytes, void* stream) {
  if (int e = check_desc(d, false)) return e;
  if (int e = check_norm(d, false)) return e;
  PQ_REQUIRE(d->w_kind == PQ_W_MASTER, PQ_ERR_BAD_ARG, "the normalising entry point takes latent weights");
  PQ_REQUIRE(X && gain && W && ctx && workspace, PQ_ERR_BAD_ARG, "NULL buffer (X, gain, W, ctx or workspace)");
  PQ_REQUIRE(eps >= 0.0f, PQ_ERR_BAD_ARG, "eps must not be negative");
  PQ_REQUIRE(aligned16(X) && aligned16(gain) && aligned16(W) && aligned16(ctx) && aligned16(workspace), PQ_ERR_SHAPE, "buffers must be 16-byte aligned");
  const lin_layout L = make_layout(*d);
  const norm_layout NL = make_norm_layout(*d, L);
  PQ_REQUIRE(ctx_bytes >= NL.ctx_total, PQ_ERR_WORKSPACE, "ctx too small: %zu < %zu", ctx_bytes, NL.ctx_total);
  PQ_REQUIRE(workspace_bytes >= NL.ws_base, PQ_ERR_WORKSPACE, "workspace too small: %zu < %zu", workspace_bytes, NL.ws_base);
  char* cx = (char*)ctx;
  const bool bf16 = d->io_dtype == PQ_BF16;
  void* Xn = cx + NL.Xn;
  const size_t n = (size_t)d->d_out * d->d_in;
  if (int e = pq_launch_rmsnorm_quant(X, gain, d->io_dtype, d->tokens, d->d_in, eps, Xn, (int8_t*)(cx + L.Xq), (float*)(cx + L.gamma),
                                      bf16 ? (uint16_t*)(cx + L.Xt) : nullptr, (float*)(cx + NL.rstd), (hipStream_t)stream, W, n,
                                      (double*)((char*)workspace + L.stat_partials), pq_stats_blocks(n)))
    return e;
  return linear_fwd_impl(d, Xn, W, nullptr, hpA, hpB, Wr, Y, ctx, L.ctx_total, workspace, L.ws_base, stream, true);
}

extern "C" int pq_linear_norm_bwd(const pq_linear_desc* d, const void* dY, const void* X, const void* gain, const void* W,
                                  const void* hpA, const void* hpB, const void* Wr, const void* ctx, size_t ctx_bytes, void* dX,
                                  float* dgain, float* dW, float* dhpA, float* dhpB, float* dWr, float* dalpha_dbeta,
                                  void* workspace, size_t workspace_bytes, void* stream) {
  if (int e = check_desc(d, true)) return e;
  if (int e = check_norm(d, true)) return e;
  PQ_REQUIRE(X && gain && ctx && dX && dgain && workspace, PQ_ERR_BAD_ARG, "NULL buffer");
  PQ_REQUIRE(aligned16(X) && aligned16(gain) && aligned16(dX) && aligned16(workspace), PQ_ERR_SHAPE, "buffers must be 16-byte aligned");
  const lin_layout L = make_layout(*d);
  const norm_layout NL = make_norm_layout(*d, L);
  PQ_REQUIRE(ctx_bytes >= NL.ctx_total, PQ_ERR_WORKSPACE, "ctx too small: %zu < %zu", ctx_bytes, NL.ctx_total);
  PQ_REQUIRE(workspace_bytes >= NL.ws_base, PQ_ERR_WORKSPACE, "workspace too small: %zu < %zu", workspace_bytes, NL.ws_base);
  const char* cx = (const char*)ctx;
  char* ws = (char*)workspace;
  void* dXn = ws + NL.dXn;
  if (int e = linear_bwd_impl(d, dY, cx + NL.Xn, W, hpA, hpB, Wr, ctx, L.ctx_total, dXn, dW, dhpA, dhpB, dWr, dalpha_dbeta, workspace,
                              L.ws_base, stream, workspace_bytes >= NL.ws_total ? ws + NL.ws_base : nullptr))
    return e;
  float* part = (float*)(((uintptr_t)(ws + NL.part) + 255) & ~(uintptr_t)255);
  return pq_launch_rmsnorm_bwd(dXn, X, gain, (const float*)(cx + NL.rstd), d->io_dtype, d->tokens, d->d_in, dX, dgain, part,
                               (hipStream_t)stream);
}

// ---------------------------------------------------------------------------------------------
// INT8 form of the two-factor high-precision branch (Sec. 3.2): rows of A and B and the hidden state are
// quantised like activations; both products run on the int8 MFMA path with exact int32 accumulation and a
// de-quantising epilogue (row scale as a reciprocal per row, column scale by division).  The backward is the
// STE one: bf16 GEMMs on the de-quantised factors saved by the forward.
// ctx: [Aq r*K][gA r][At r*K bf16][Bq N*r][gB N][Bt N*r bf16][H T*r bf16][Hq T*r][gH T][Ht T*r bf16]
// workspace: [dH T*r bf16][split-contraction slabs]
// ---------------------------------------------------------------------------------------------
namespace {
int check_hp8(int dtype, int T, int K, int N, int r) {
  PQ_REQUIRE(dtype == PQ_BF16, PQ_ERR_DTYPE, "the INT8 high-precision branch takes bf16 tensors");
  PQ_REQUIRE(T >= 0 && K > 0 && N > 0 && r > 0, PQ_ERR_BAD_ARG, "bad size T=%d K=%d N=%d r=%d", T, K, N, r);
  PQ_REQUIRE(K % 32 == 0 && N % 32 == 0 && r % 32 == 0, PQ_ERR_SHAPE, "K=%d, N=%d and r=%d must be multiples of 32", K, N, r);
  return PQ_OK;
}
}  // namespace

extern "C" size_t pq_hp_int8_ctx_bytes(int32_t T, int32_t K, int32_t N, int32_t r) {
  if (check_hp8(PQ_BF16, T, K, N, r) != PQ_OK) return 0;
  return make_hp8_layout(T, K, N, r).ctx_total;
}
extern "C" size_t pq_hp_int8_workspace_bytes(int32_t T, int32_t K, int32_t N, int32_t r) {
  if (check_hp8(PQ_BF16, T, K, N, r) != PQ_OK) return 0;
  return make_hp8_layout(T, K, N, r).ws_total;
}

extern "C" int pq_hp_int8_fwd(const int8_t* Xq, const float* gamma_x, const void* A, const void* B, int32_t dtype, int32_t T,
                              int32_t K, int32_t N, int32_t r, float alpha, void* Y, int32_t accumulate, void* ctx,
                              size_t ctx_bytes, void* workspace, size_t workspace_bytes, void* stream) {
  return hp_int8_fwd_impl(Xq, gamma_x, A, B, dtype, T, K, N, r, alpha, Y, accumulate, ctx, ctx_bytes, workspace, workspace_bytes, stream, false);
}

static int hp_int8_fwd_impl(const int8_t* Xq, const float* gamma_x, const void* A, const void* B, int32_t dtype, int32_t T, int32_t K,
                            int32_t N, int32_t r, float alpha, void* Y, int32_t accumulate, void* ctx, size_t ctx_bytes, void* workspace,
                            size_t workspace_bytes, void* stream, bool rows_done) {
  if (int e = check_hp8(dtype, T, K, N, r)) return e;
  const hp8_layout L = make_hp8_layout(T, K, N, r);
  PQ_REQUIRE(A && B && ctx && workspace, PQ_ERR_BAD_ARG, "NULL buffer (A, B, ctx or workspace)");
  PQ_REQUIRE(T == 0 || (Xq && gamma_x && Y), PQ_ERR_BAD_ARG, "NULL buffer (Xq, gamma_x or Y)");
  PQ_REQUIRE(aligned16(Xq) && aligned16(A) && aligned16(B) && aligned16(Y) && aligned16(ctx) && aligned16(workspace), PQ_ERR_SHAPE,
             "buffers must be 16-byte aligned");
  PQ_REQUIRE(ctx_bytes >= L.ctx_total, PQ_ERR_WORKSPACE, "ctx too small: %zu < %zu", ctx_bytes, L.ctx_total);
  PQ_REQUIRE(workspace_bytes >= L.ws_total, PQ_ERR_WORKSPACE, "workspace too small: %zu < %zu", workspace_bytes, L.ws_total);
  hipStream_t s = (hipStream_t)stream;
  char* cx = (char*)ctx;
  const pq_scratch sk{(char*)workspace + L.splitk, L.splitk_bytes};
  // weight side: rows of A and B on the activation grid (codes, gamma, bf16 de-quantised copy for the backward)
  if (!rows_done) {
    if (int e = pq_launch_quant_act(A, dtype, r, K, (int8_t*)(cx + L.Aq), (float*)(cx + L.gA), (uint16_t*)(cx + L.At), s)) return e;
    if (int e = pq_launch_quant_act(B, dtype, N, r, (int8_t*)(cx + L.Bq), (float*)(cx + L.gB), (uint16_t*)(cx + L.Bt), s)) return e;
  }
  if (T == 0) return PQ_OK;
  {  // H = (q_x q_a^T) / (gamma_x gamma_a)
    pq_operand a{Xq, K, PQ_SRC_KC8, nullptr};
    pq_operand b{cx + L.Aq, K, PQ_SRC_KC8, nullptr};
    pq_epilogue e = epi_zero();
    e.C = cx + L.H; e.ldc = r; e.out_kind = PQ_OUT_BF16; e.row_div = gamma_x; e.col_div = (const float*)(cx + L.gA);
    e.split_int8 = 1;
    if (int err = pq_launch_gemm(T, r, K, a, b, e, s, PQP_GEMM_HP_H, sk)) return err;
  }
  if (int e = pq_launch_quant_act(cx + L.H, dtype, T, r, (int8_t*)(cx + L.Hq), (float*)(cx + L.gH), (uint16_t*)(cx + L.Ht), s)) return e;
  {  // Y (+)= alpha * (q_h q_b^T) / (gamma_h gamma_b)
    pq_operand a{cx + L.Hq, r, PQ_SRC_KC8, nullptr};
    pq_operand b{cx + L.Bq, r, PQ_SRC_KC8, nullptr};
    pq_epilogue e = epi_zero();
    e.C = Y; e.ldc = N; e.out_kind = PQ_OUT_BF16; e.accumulate = accumulate ? 1 : 0; e.scale = alpha;
    e.row_div = (const float*)(cx + L.gH); e.col_div = (const float*)(cx + L.gB);
    if (int err = pq_launch_gemm(T, N, r, a, b, e, s, PQP_GEMM_HP_Y, sk)) return err;
  }
  return PQ_OK;
}

extern "C" int pq_hp_int8_bwd(const void* dY, const void* Xt, int32_t dtype, int32_t T, int32_t K, int32_t N, int32_t r,
                              float alpha, const void* ctx, size_t ctx_bytes, void* dX, int32_t accumulate_dX, float* dA, float* dB,
                              void* workspace, size_t workspace_bytes, void* stream) {
  if (int e = check_hp8(dtype, T, K, N, r)) return e;
  const hp8_layout L = make_hp8_layout(T, K, N, r);
  PQ_REQUIRE(ctx && dA && dB && workspace, PQ_ERR_BAD_ARG, "NULL buffer (ctx, dA, dB or workspace)");
  PQ_REQUIRE(T == 0 || (dY && Xt && dX), PQ_ERR_BAD_ARG, "NULL buffer (dY, Xt or dX)");
  PQ_REQUIRE(aligned16(dY) && aligned16(Xt) && aligned16(ctx) && aligned16(dX) && aligned16(dA) && aligned16(dB) && aligned16(workspace),
             PQ_ERR_SHAPE, "buffers must be 16-byte aligned");
  PQ_REQUIRE(ctx_bytes >= L.ctx_total, PQ_ERR_WORKSPACE, "ctx too small: %zu < %zu", ctx_bytes, L.ctx_total);
  PQ_REQUIRE(workspace_bytes >= L.ws_total, PQ_ERR_WORKSPACE, "workspace too small: %zu < %zu", workspace_bytes, L.ws_total);
  hipStream_t s = (hipStream_t)stream;
  const char* cx = (const char*)ctx;
  char* ws = (char*)workspace;
  if (T > 0)
    if (int e = hp_int8_dh(dY, T, N, r, alpha, cx, L, ws, nullptr, s)) return e;
  if (int e = hp_int8_factor_grads(dY, Xt, T, K, N, r, alpha, cx, L, dA, dB, ws, nullptr, nullptr, s, nullptr)) return e;
  if (T > 0) {  // dX (+)= dH A~
    pq_operand a{ws + L.dH, r, PQ_SRC_KC16, nullptr};
    pq_operand b{cx + L.At, K, PQ_SRC_KS16, nullptr};
    pq_epilogue e = epi_zero();
    e.C = dX; e.ldc = K; e.out_kind = PQ_OUT_BF16; e.accumulate = accumulate_dX ? 1 : 0;
    if (int err = pq_launch_gemm(T, K, r, a, b, e, s, PQP_GEMM_DX_HP, {ws + L.splitk, L.splitk_bytes})) return err;
  }
  return PQ_OK;
}

static int hp_int8_dh(const void* dY, int T, int N, int r, float alpha, const char* cx, const hp8_layout& L, char* ws, double* red_a, hipStream_t s) {
  pq_operand a{dY, N, PQ_SRC_KC16, nullptr};
  pq_operand b{cx + L.Bt, r, PQ_SRC_KS16, nullptr};
  pq_epilogue e = epi_zero();
  e.C = ws + L.dH; e.ldc = r; e.out_kind = PQ_OUT_BF16; e.scale = alpha;
  if (red_a) {   // sum H~ .* (dY B~) = <dY, H~ B~^T>
    e.dot_comp = cx + L.Ht; e.ld_comp = r; e.comp_kind = PQ_OUT_BF16; e.partials = red_a;
  }
  return pq_launch_gemm(T, r, N, a, b, e, s, PQP_GEMM_DH, {ws + L.splitk, L.splitk_bytes});
}

static int hp_int8_factor_grads(const void* dY, const void* Xt, int T, int K, int N, int r, float alpha, const char* cx, const hp8_layout& L,
                                float* dA, float* dB, char* ws, const pq_reduce_job* jobs, bool* jobs_done, hipStream_t s,
                                const pq_grads* along) {
  // dB = alpha * dY^T H~ and dA = dH^T X~ (dH already carries alpha): one launch when their shapes allow it
  const void* dH = ws + L.dH;
  pq_operand a0{dY, N, PQ_SRC_KS16, nullptr}, b0{cx + L.Ht, r, PQ_SRC_KS16, nullptr};
  pq_operand a1{dH, r, PQ_SRC_KS16, nullptr}, b1{Xt, K, PQ_SRC_KS16, nullptr};
  return pq_launch_gemm_pair_ks16(T, N, r, a0, b0, dB, r, alpha, r, K, a1, b1, dA, K, 1.0f, s, PQP_GEMM_DB, PQP_GEMM_DA, {ws + L.splitk, L.splitk_bytes},
                                  {ws + L.splitk2, L.splitk2_bytes}, jobs, jobs_done, along);
}

// ---------------------------------------------------------------------------------------------
// Decode on packed weights
// ---------------------------------------------------------------------------------------------
namespace {
int check_decode(const pq_decode_desc* d) {
  PQ_REQUIRE(d != nullptr, PQ_ERR_BAD_ARG, "desc is NULL");
  PQ_REQUIRE(d->batch >= 1 && d->batch <= 16, PQ_ERR_BAD_ARG, "batch=%d must be in 1..16", d->batch);
  PQ_REQUIRE(d->d_in > 0 && d->d_out > 0 && d->hp_rank >= 0 && d->n_layers >= 1, PQ_ERR_BAD_ARG, "bad dimension");
  PQ_REQUIRE(d->d_out % 4 == 0, PQ_ERR_SHAPE, "d_out=%d must be a multiple of 4", d->d_out);
  PQ_REQUIRE(d->d_in <= 16384, PQ_ERR_SHAPE, "d_in=%d exceeds 16384 (one token's activations are staged in LDS)", d->d_in);
  PQ_REQUIRE(d->packed_layout == PQ_PACKED_ROWMAJOR || d->packed_layout == PQ_PACKED_TILED64, PQ_ERR_BAD_ARG,
             "packed_layout=%d is not a known layout", d->packed_layout);
  const bool tiled = d->packed_layout == PQ_PACKED_TILED64;
  if (d->batch == 1) {
    PQ_REQUIRE(d->d_in % 128 == 0, PQ_ERR_SHAPE, "d_in=%d must be a multiple of 128", d->d_in);
    PQ_REQUIRE(d->hp_rank % 8 == 0, PQ_ERR_SHAPE, "hp_rank=%d must be a multiple of 8", d->hp_rank);
  } else {
    if (tiled) PQ_REQUIRE(d->d_in % 128 == 0, PQ_ERR_SHAPE, "d_in=%d must be a multiple of 128", d->d_in);
    else PQ_REQUIRE(d->d_in % 512 == 0, PQ_ERR_SHAPE, "batch > 1 on the row-major packing needs d_in=%d to be a multiple of 512", d->d_in);
    PQ_REQUIRE(d->hp_rank % 32 == 0, PQ_ERR_SHAPE, "batch > 1 needs hp_rank=%d to be a multiple of 32", d->hp_rank);
  }
  if (d->hp_rank > 0) {
    PQ_REQUIRE(d->n_experts >= 1 && d->n_experts <= 64, PQ_ERR_BAD_ARG, "n_experts=%d must be in 1..64", d->n_experts);
    PQ_REQUIRE(d->top_k >= 1 && d->top_k <= d->n_experts, PQ_ERR_BAD_ARG, "top_k=%d must be in 1..n_experts", d->top_k);
    if (d->batch > 1) PQ_REQUIRE((d->n_experts * d->hp_rank) % 64 == 0, PQ_ERR_SHAPE, "batch > 1 needs n_experts*hp_rank %% 64 == 0");
  }
  if (d->batch > 1) {
    // LDS of the small-batch kernels: 8 or 16 token rows of codes and expert hidden states; on the
    // row-interleaved packing the hidden states share their space with 8 KiB of per-wavefront patches
    const size_t toks = d->batch <= 8 ? 8 : 16;
    const size_t er = d->hp_rank > 0 ? (size_t)d->n_experts * d->hp_rank : 0;
    const size_t hm = 2 * toks * er;
    // (the row-interleaved kernel walks the codes in blocks of 32 KiB)
    const size_t codes = tiled && toks * (size_t)d->d_in > 32768 ? 32768 : toks * (size_t)d->d_in;
    PQ_REQUIRE(codes + ((tiled && hm < 8192) ? 8192 : hm) <= 160 * 1024, PQ_ERR_SHAPE,
               "activations and expert hidden states do not fit the 160 KiB LDS");
  }
  return PQ_OK;
}
}  // namespace

extern "C" size_t pq_decode_workspace_bytes(const pq_decode_desc* d) {
  if (check_decode(d) != PQ_OK) return 0;
  pq_decode_desc dd = *d;
  if (dd.hp_rank == 0) dd.top_k = 0;
  size_t off[7];
  return pq_decode_ws_layout(dd, off);
}

extern "C" int pq_decode_gemv(const pq_decode_desc* d, const void* X, const uint32_t* packed, const uint16_t* scale_fp16,
                              const void* hpA, const void* hpB, const void* Wr, void* Y, int32_t* acc_out, void* workspace,
                              size_t workspace_bytes, void* stream) {
  if (int e = check_decode(d)) return e;
  PQ_REQUIRE(X && packed && scale_fp16 && Y && workspace, PQ_ERR_BAD_ARG, "NULL buffer");
  PQ_REQUIRE(d->hp_rank == 0 || (hpA && hpB && Wr), PQ_ERR_BAD_ARG, "hp_rank=%d but an expert buffer is NULL", d->hp_rank);
  PQ_REQUIRE(aligned16(X) && aligned16(packed) && aligned16(Y) && aligned16(workspace) && aligned16(hpA) && aligned16(hpB) &&
                 aligned16(Wr) && aligned16(acc_out), PQ_ERR_SHAPE, "buffers must be 16-byte aligned");
  pq_decode_desc dd = *d;
  if (dd.hp_rank == 0) dd.top_k = 0;
  size_t off[7];
  const size_t need = pq_decode_ws_layout(dd, off);
  PQ_REQUIRE(workspace_bytes >= need, PQ_ERR_WORKSPACE, "workspace too small: %zu < %zu", workspace_bytes, need);
  return pq_launch_decode(dd, X, packed, scale_fp16, hpA, hpB, Wr, Y, acc_out, workspace, (hipStream_t)stream);
}

extern "C" int pq_decode_gemv_int8(const pq_decode_desc* d, const void* X, const uint32_t* packed, const uint16_t* scale_fp16,
                                   const int8_t* hpA_q, const float* gamma_A, const int8_t* hpB_q, const float* gamma_B,
                                   const void* Wr, void* Y, int32_t* acc_out, void* workspace, size_t workspace_bytes,
                                   void* stream) {
  if (int e = check_decode(d)) return e;
  PQ_REQUIRE(d->hp_rank > 0 && d->hp_rank % 32 == 0, PQ_ERR_SHAPE, "hp_rank=%d must be a positive multiple of 32", d->hp_rank);
  if (d->batch == 1) {
    PQ_REQUIRE(d->top_k <= 8 && d->top_k * d->hp_rank <= 2048, PQ_ERR_SHAPE, "top_k=%d (at most 8) times hp_rank=%d exceeds 2048",
               d->top_k, d->hp_rank);
    PQ_REQUIRE((size_t)d->d_in * 5 <= 64 * 1024, PQ_ERR_SHAPE, "d_in=%d exceeds 13056 (activations and their codes are staged in LDS)", d->d_in);
  } else {
    PQ_REQUIRE(d->packed_layout == PQ_PACKED_TILED64, PQ_ERR_SHAPE, "INT8 experts with batch > 1 need the row-interleaved packing");
    PQ_REQUIRE(d->hp_rank % 64 == 0 && (d->n_experts * d->hp_rank) % 128 == 0, PQ_ERR_SHAPE,
               "INT8 experts with batch > 1 need hp_rank=%d %% 64 == 0 and n_experts * hp_rank %% 128 == 0", d->hp_rank);
    PQ_REQUIRE(d->d_out % 4 == 0, PQ_ERR_SHAPE, "d_out=%d must be a multiple of 4", d->d_out);
  }
  PQ_REQUIRE(X && packed && scale_fp16 && Y && workspace && hpA_q && gamma_A && hpB_q && gamma_B && Wr, PQ_ERR_BAD_ARG, "NULL buffer");
  PQ_REQUIRE(aligned16(X) && aligned16(packed) && aligned16(Y) && aligned16(workspace) && aligned16(hpA_q) && aligned16(hpB_q) &&
                 aligned16(Wr) && aligned16(acc_out), PQ_ERR_SHAPE, "buffers must be 16-byte aligned");
  size_t off[7];
  const size_t need = pq_decode_ws_layout(*d, off);
  PQ_REQUIRE(workspace_bytes >= need, PQ_ERR_WORKSPACE, "workspace too small: %zu < %zu", workspace_bytes, need);
  return pq_launch_decode(*d, X, packed, scale_fp16, hpA_q, hpB_q, Wr, Y, acc_out, workspace, (hipStream_t)stream, gamma_A, gamma_B);
}

// ---------------------------------------------------------------------------------------------
// Decoupled FFN at inference: workspace = [decode workspace of the up/gate stage (rank 2r)][U and G, 2 L F bf16]
// [decode workspace of the down stage]
// ---------------------------------------------------------------------------------------------
namespace {
struct dffn_layout { size_t ws1, UG, ws2, amax, total; };
int check_dffn(const pq_decode_ffn_desc* d) {
  PQ_REQUIRE(d != nullptr, PQ_ERR_BAD_ARG, "desc is NULL");
  PQ_REQUIRE(d->d_model > 0 && d->d_ffn > 0 && d->hp_rank > 0 && d->n_layers >= 1, PQ_ERR_BAD_ARG, "bad dimension");
  PQ_REQUIRE(d->d_model % 128 == 0 && d->d_ffn % 128 == 0, PQ_ERR_SHAPE, "d_model=%d and d_ffn=%d must be multiples of 128", d->d_model, d->d_ffn);
  PQ_REQUIRE(d->d_model <= 16384 && d->d_ffn <= 16384, PQ_ERR_SHAPE, "d_model=%d / d_ffn=%d exceed 16384 (a token's activations are staged in LDS)", d->d_model, d->d_ffn);
  PQ_REQUIRE(d->hp_rank % 8 == 0, PQ_ERR_SHAPE, "hp_rank=%d must be a multiple of 8", d->hp_rank);
  PQ_REQUIRE(d->n_experts >= 1 && d->n_experts <= 64, PQ_ERR_BAD_ARG, "n_experts=%d must be in 1..64", d->n_experts);
  PQ_REQUIRE(d->top_k >= 1 && d->top_k <= d->n_experts, PQ_ERR_BAD_ARG, "top_k=%d must be in 1..n_experts", d->top_k);
  PQ_REQUIRE(d->batch >= 0 && d->batch <= 16, PQ_ERR_BAD_ARG, "batch=%d must be in 1..16 (0 stands for 1)", d->batch);
  if (d->batch > 1) {
    PQ_REQUIRE(d->hp_rank % 32 == 0 && (d->n_experts * d->hp_rank) % 64 == 0, PQ_ERR_SHAPE,
               "batch > 1 needs hp_rank=%d %% 32 == 0 and n_experts * hp_rank %% 64 == 0", d->hp_rank);
    // LDS of the small-batch kernels: a block of the 8 or 16 token rows of codes, and for the down product the expert hidden states
    const size_t toks = d->batch <= 8 ? 8 : 16;
    const size_t hm = 2 * toks * (size_t)d->n_experts * d->hp_rank;
    PQ_REQUIRE(32768 + (hm < 8192 ? 8192 : hm) <= 160 * 1024, PQ_ERR_SHAPE,
               "expert hidden states of %d tokens do not fit the 160 KiB LDS next to a 32 KiB block of codes", d->batch);
  }
  return PQ_OK;
}
dffn_layout make_dffn_layout(const pq_decode_ffn_desc& d) {
  const int B = d.batch > 1 ? d.batch : 1;
  pq_decode_desc d1{B, d.d_model, d.d_ffn, 2 * d.hp_rank, d.n_experts, d.top_k, d.n_layers, PQ_PACKED_TILED64, d.alpha};
  pq_decode_desc d2{B, d.d_ffn, d.d_model, d.hp_rank, d.n_experts, d.top_k, d.n_layers, PQ_PACKED_TILED64, d.alpha};
  size_t off[7];
  dffn_layout L;
  cursor c;
  L.ws1 = c.take(pq_decode_ws_layout(d1, off));
  L.UG = c.take((size_t)2 * d.n_layers * B * d.d_ffn * 2);
  L.ws2 = c.take(pq_decode_ws_layout(d2, off));
  // maxima of the gated hidden state: of a token's eight parts, at one token per layer of 64 columns each
  L.amax = c.take((size_t)d.n_layers * (B > 1 ? B * 8 : (d.d_ffn + 63) / 64) * sizeof(float));
  L.total = c.off;
  return L;
}
}  // namespace

extern "C" size_t pq_decode_ffn_workspace_bytes(const pq_decode_ffn_desc* d) {
  if (check_dffn(d) != PQ_OK) return 0;
  return make_dffn_layout(*d).total;
}

extern "C" int pq_decode_ffn(const pq_decode_ffn_desc* d, const void* X, const uint32_t* packed_upgate, const uint16_t* scale_upgate,
                             const uint32_t* packed_down, const uint16_t* scale_down, const void* UpGate, const void* Down,
                             const void* Wr, void* Y, int32_t* acc_upgate, void* workspace, size_t workspace_bytes, void* stream) {
  if (int e = check_dffn(d)) return e;
  PQ_REQUIRE(X && packed_upgate && scale_upgate && packed_down && scale_down && UpGate && Down && Wr && Y && workspace, PQ_ERR_BAD_ARG,
             "NULL buffer");
  PQ_REQUIRE(aligned16(X) && aligned16(packed_upgate) && aligned16(packed_down) && aligned16(UpGate) && aligned16(Down) && aligned16(Wr) &&
                 aligned16(Y) && aligned16(acc_upgate) && aligned16(workspace), PQ_ERR_SHAPE, "buffers must be 16-byte aligned");
  const dffn_layout L = make_dffn_layout(*d);
  PQ_REQUIRE(workspace_bytes >= L.total, PQ_ERR_WORKSPACE, "workspace too small: %zu < %zu", workspace_bytes, L.total);
  char* ws = (char*)workspace;
  return pq_launch_decode_ffn(d->n_layers, d->batch > 1 ? d->batch : 1, d->d_model, d->d_ffn, d->hp_rank, d->n_experts, d->top_k, d->alpha, X, packed_upgate,
                              scale_upgate, packed_down, scale_down, UpGate, Down, Wr, Y, acc_upgate, ws + L.UG, ws + L.ws1, ws + L.ws2,
                              (float*)(ws + L.amax), (hipStream_t)stream);
}

extern "C" size_t pq_pack_tiled64_bytes(int32_t N, int32_t K) {
  if (N <= 0 || K <= 0 || K % 128 != 0) return 0;
  return (size_t)((N + 63) / 64) * 64 * (K / 32) * sizeof(uint32_t);
}

extern "C" int pq_pack_retile64(const uint32_t* packed, int32_t N, int32_t K, uint32_t* tiled, void* stream) {
  PQ_REQUIRE(N > 0 && K > 0, PQ_ERR_BAD_ARG, "bad size N=%d K=%d", N, K);
  PQ_REQUIRE(K % 128 == 0, PQ_ERR_SHAPE, "K=%d must be a multiple of 128", K);
  PQ_REQUIRE(packed && tiled, PQ_ERR_BAD_ARG, "NULL buffer");
  PQ_REQUIRE(aligned16(packed) && aligned16(tiled), PQ_ERR_SHAPE, "buffers must be 16-byte aligned");
  return pq_launch_retile64(packed, N, K, tiled, (hipStream_t)stream);
}

// ---------------------------------------------------------------------------------------------
// Glue for chaining linears into a layer stack (not part of the method: residual adds, row gather)
// ---------------------------------------------------------------------------------------------
extern "C" int pq_glue_lincomb(void* out, const void* x0, const void* x1, const void* x2, const void* x3, float c0,
                               float c1, float c2, float c3, size_t n, void* stream) {
  PQ_REQUIRE(out && x0, PQ_ERR_BAD_ARG, "NULL buffer");
  PQ_REQUIRE(n % 8 == 0, PQ_ERR_SHAPE, "n=%zu must be a multiple of 8", n);
  PQ_REQUIRE(aligned16(out) && aligned16(x0) && aligned16(x1) && aligned16(x2) && aligned16(x3), PQ_ERR_SHAPE,
             "buffers must be 16-byte aligned");
  return pq_launch_lincomb(out, x0, x1, x2, x3, c0, c1, c2, c3, n, (hipStream_t)stream);
}

extern "C" int pq_glue_gather_rows(const void* table, const int32_t* ids, int32_t T, int32_t d, void* out, void* stream) {
  PQ_REQUIRE(T >= 0 && d > 0 && d % 8 == 0, PQ_ERR_SHAPE, "bad shape T=%d d=%d (d must be a multiple of 8)", T, d);
  if (T == 0) return PQ_OK;
  PQ_REQUIRE(table && ids && out, PQ_ERR_BAD_ARG, "NULL buffer");
  PQ_REQUIRE(aligned16(table) && aligned16(out), PQ_ERR_SHAPE, "buffers must be 16-byte aligned");
  return pq_launch_gather_rows(table, ids, 1, T, d, out, (hipStream_t)stream);
}
