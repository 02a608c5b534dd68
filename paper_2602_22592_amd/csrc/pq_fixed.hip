// fp32 I/O, large products: the two big contractions of the backward, dX = dY S and dW = (dY / gamma)^T q, as exact integer
// products on the int8 matrix pipe.
//
// One operand of each is already small integers (signs, codes), so only dY has to be cut up: a row of the left operand (a
// token of dY, or an output channel over the tokens) is written as fixed-point numbers of 55 bits relative to its largest
// element, X = rint(x 2^(54 - E)), max |x| < 2^E, and those as seven signed digits of base 256, each a plane of int8 (the
// splitting of operands into slices whose products are exact: Ozaki, Ogita, Oishi, Rump, "Error-free transformations of matrix
// multiplication", 2012).  Seven int8 products with int32 sums are exact; their sum sum_d 256^d acc_d 2^(E - 54) is formed in fp64
// (pq_ref.hip, the SUM forms).  What is lost is the rounding of an element to 2^(E - 55).  In dX every element of a row enters every
// sum, and the additions behind the largest one round as much in fp64.  In dW a token whose code is zero stays out of a sum, and the
// largest element may be such a token's.  The column pass therefore counts the small elements, below 2^(E - 17), the zero ones and,
// per channel, the zero codes; a sum is taken from the planes only if, with l = tokens - small - zero ones and z the zero codes,
//     8 max(l - z, 0) >= min(small, tokens - z):
// at least l - z larger elements enter it then and at most eight times as many small ones, so that it is off by at most 2^-28 of
// sum |x q|, a sixteenth of the rounding to fp32.  A 32x32 tile with another sum in it
// is formed as the fp64 product it stands for.  One token 1e9 / 1e12 / 1e16 times the others: relative error of the sums that its zero
// codes leave out 3.2e-8 / 1.9e-5 / 0.2 from the planes, 2.6e-8 now.  Backward of 2048 tokens 2048x2048 (us): 248 with normal data; 218 to
// 249 with 95 % zero codes, half of the tokens masked, token scales of e^+-6 or elements of e^+-10; 538 with one token 1e6 times the others
// (all tiles fp64).
// What it is for: the fp64 matrix rate is 78.6 TFLOP/s, the int8 one 5 POP/s nominal and 2 on real data, so seven products cost a
// quarter of one fp64 product.  2048 tokens, 2048x2048, r = 128 (us): dX 277 -> 74 + 55 (with the rank-128 product and dA), dW 275 -> 77 + 63 (with
// dB and dH); the passes below 13, 5 and 20, two of them over dY, 4 bytes read and 7 written per element; whole step 718 -> 380.
// Infinities and NaN have no fixed-point form: their rows get no digits and are marked, and the SUM forms compute a 32x32 tile that
// a marked row reaches as the fp64 product it stands for.  Step of 2048 tokens 2048x2048 (us): finite 300; one NaN in dY 443; an infinity in X, which marks every
// row of dW, 604 (one element after the other: 1115 and 5368; fp64 products alone 600).
#include <string.h>
#include "pq_internal.h"

namespace {

constexpr int ND = PQ_FIXED_DIGITS;
constexpr int COLT = 128;                            // tokens per workgroup of the column pass
constexpr int SMALL = 37;                            // digits below 2^37: elements below 2^(E - 17)
constexpr int ROWS = 8;                              // rows of dY per workgroup of the row pass, four to a half of it

// 1 / gamma in fp64, as the fp64 products form it (pq_ref.hip)
__device__ __forceinline__ double recip(float g) {
  const double d = (double)g;
  double r = __builtin_amdgcn_rcp(d);
  r = __builtin_fma(r, __builtin_fma(-d, r, 1.0), r);
  return __builtin_fma(r, __builtin_fma(-d, r, 1.0), r);
}

__device__ __forceinline__ double pow2(int e) { return __builtin_bit_cast(double, (uint64_t)(e + 1023) << 52); }   // normal range

// the seven digits of rint(v) (|v| <= 2^54) in the bytes of a 64-bit word, lowest first: adding 128 to every digit but the top one
// carries what a signed digit borrows, and leaves each byte off by the 128 that the exclusive or takes back
__device__ __forceinline__ uint64_t digits(double v) {
  const uint64_t x = (uint64_t)(int64_t)__builtin_rint(v) + 0x0000808080808080ull;
  return x ^ 0x0000808080808080ull;
}

// Bytes d of four digit words as one word, for every d: two 4x4 byte transposes (the eighth byte is not used).
__device__ __forceinline__ void planes_of(const uint64_t (&w)[4], uint32_t (&o)[ND]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t a = (uint32_t)(w[0] >> (32 * h)), b = (uint32_t)(w[1] >> (32 * h)), c = (uint32_t)(w[2] >> (32 * h)), d = (uint32_t)(w[3] >> (32 * h));
    const uint32_t ab0 = __builtin_amdgcn_perm(b, a, 0x05010400u), ab1 = __builtin_amdgcn_perm(b, a, 0x07030602u);   // a0 b0 a1 b1, a2 b2 a3 b3
    const uint32_t cd0 = __builtin_amdgcn_perm(d, c, 0x05010400u), cd1 = __builtin_amdgcn_perm(d, c, 0x07030602u);
    o[4 * h] = __builtin_amdgcn_perm(cd0, ab0, 0x05040100u);
    o[4 * h + 1] = __builtin_amdgcn_perm(cd0, ab0, 0x07060302u);
    o[4 * h + 2] = __builtin_amdgcn_perm(cd1, ab1, 0x05040100u);
    if (4 * h + 3 < ND) o[4 * h + 3] = __builtin_amdgcn_perm(cd1, ab1, 0x07060302u);
  }
}

// exponent E with max < 2^E from the largest |x| as bits (float), or the marker of a row that is not finite
__device__ __forceinline__ int exp_f32(uint32_t u) { return u >= 0x7F800000u ? PQ_FIXED_NOT_FINITE : max((int)(u >> 23), 1) - 126; }
// the same from the upper half of a double's bits
__device__ __forceinline__ int exp_f64(uint32_t u) { return u >= 0x7FF00000u ? PQ_FIXED_NOT_FINITE : max((int)(u >> 20), 1) - 1022; }

// Rows of dY: digits [ND][T][N] and exponents [T]; colmax [ceil(T / ROWS)][N]: the largest |dY / gamma| of the workgroup's rows, as
// the upper half of the double.  counts: cleared for the column pass.
__global__ __launch_bounds__(512) void fixed_rows_kernel(const float* __restrict__ dY, const float* __restrict__ gamma, int T, int N,
                                                         int8_t* __restrict__ D, int* __restrict__ rexp, uint32_t* __restrict__ colmax,
                                                         int* __restrict__ counts, int ncounts) {
  for (int i = blockIdx.x * 512 + threadIdx.x; i < ncounts; i += gridDim.x * 512) counts[i] = 0;
  constexpr int R = ROWS / 2;
  __shared__ uint32_t wmax[8][R];
  __shared__ uint4 cmax[256];
  const int tid = threadIdx.x & 255, half = threadIdx.x >> 8, t0 = blockIdx.x * ROWS + half * R;
  uint32_t rm[R];
  double rg[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    rm[r] = 0u;
    rg[r] = recip(gamma[min(t0 + r, T - 1)]);
  }
  for (int c0 = 0; c0 < N; c0 += 1024) {             // (N % 32 == 0; rows and columns past the end repeat the last ones)
    const int c = min(c0 + 4 * tid, N - 4);
    float4 v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = *reinterpret_cast<const float4*>(dY + (size_t)min(t0 + r, T - 1) * N + c);
    uint32_t cm[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const float x[4] = {v[r].x, v[r].y, v[r].z, v[r].w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        rm[r] = max(rm[r], __float_as_uint(x[j]) & 0x7FFFFFFFu);
        cm[j] = max(cm[j], (uint32_t)(__builtin_bit_cast(uint64_t, (double)x[j] * rg[r]) >> 32) & 0x7FFFFFFFu);
      }
    }
    if (half) cmax[tid] = make_uint4(cm[0], cm[1], cm[2], cm[3]);
    __syncthreads();
    if (!half) {
      const uint4 o = cmax[tid];
      *reinterpret_cast<uint4*>(colmax + (size_t)blockIdx.x * N + c) = make_uint4(max(cm[0], o.x), max(cm[1], o.y), max(cm[2], o.z), max(cm[3], o.w));
    }
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) rm[r] = max(rm[r], (uint32_t)__shfl_xor((int)rm[r], o, 64));
    if ((tid & 63) == 0) wmax[threadIdx.x >> 6][r] = rm[r];
  }
  __syncthreads();
  int e[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    e[r] = exp_f32(max(max(wmax[4 * half][r], wmax[4 * half + 1][r]), max(wmax[4 * half + 2][r], wmax[4 * half + 3][r])));
    if (tid == 0 && t0 + r < T) rexp[t0 + r] = e[r];
  }
  for (int c = 4 * tid; c < N; c += 1024) {
    float4 v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = *reinterpret_cast<const float4*>(dY + (size_t)min(t0 + r, T - 1) * N + c);   // (from the caches)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (t0 + r >= T) break;                        // uniform for the wavefront
      const bool ok = e[r] != PQ_FIXED_NOT_FINITE;
      const double s = ok ? pow2(54 - e[r]) : 0.0;
      const uint64_t w[4] = {ok ? digits((double)v[r].x * s) : 0, ok ? digits((double)v[r].y * s) : 0, ok ? digits((double)v[r].z * s) : 0,
                             ok ? digits((double)v[r].w * s) : 0};
      uint32_t o[ND];
      planes_of(w, o);
#pragma unroll
      for (int d = 0; d < ND; ++d) *reinterpret_cast<uint32_t*>(D + ((size_t)d * T + t0 + r) * N + c) = o[d];
    }
  }
}

// Exponents [N] of the columns of dY / gamma from the nmax rows of colmax.  (Every workgroup of the pass below
// reducing its own columns was T / 128 times these reads, quadratic in the tokens: step of 65536 tokens 512x512 1710 us, now 1274; of 2048
// tokens 2048x2048 0.8 us less than with this launch.)
__global__ __launch_bounds__(1024) void fixed_exps_kernel(const uint32_t* __restrict__ colmax, int nmax, int N, int* __restrict__ cexp) {
  __shared__ uint32_t wmax[16][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, n = blockIdx.x * 64 + lane, nc = min(n, N - 1);
  uint32_t m = 0u;
  for (int b = wv; b < nmax; b += 256) {             // sixteen requests in flight
    uint32_t x[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) x[u] = colmax[(size_t)min(b + 16 * u, nmax - 1) * N + nc];
#pragma unroll
    for (int u = 0; u < 16; ++u) m = max(m, x[u]);
  }
  wmax[wv][lane] = m;
  __syncthreads();
  if (wv > 0 || n >= N) return;
#pragma unroll
  for (int w = 1; w < 16; ++w) m = max(m, wmax[w][lane]);
  cexp[n] = exp_f64(m);
}

// Columns of dY / gamma over the tokens: digits [ND][N][Tp]; and q transposed, [K][Tp].  Tp: T rounded up to whole
// 16 bytes, the rest zero.  counts: small elements [N], zero ones [N], zero codes [K].  Workgroups (column block, token block of COLT): N / 64 of digits, then K / 256 of codes.
__global__ __launch_bounds__(256) void fixed_cols_kernel(const float* __restrict__ dY, const float* __restrict__ gamma, const int8_t* __restrict__ q,
                                                         int T, int Tp, int N, int K, const int* __restrict__ cexp, int8_t* __restrict__ D,
                                                         int8_t* __restrict__ qT, int* __restrict__ counts, int nblk) {
  __shared__ int zero_codes[256];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if ((int)blockIdx.x >= nblk) {                     // uniform: four columns of codes per lane, sixteen tokens per wavefront
    const int k0 = ((int)blockIdx.x - nblk) * 256, k = k0 + 4 * lane;
    zero_codes[threadIdx.x] = 0;
    __syncthreads();
    const int tend = k < K ? min(Tp, (int)(blockIdx.y + 1) * COLT) : 0;
    for (int t0 = blockIdx.y * COLT + wv * 16; t0 < tend; t0 += 64) {
      uint32_t w[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) w[i] = *reinterpret_cast<const uint32_t*>(q + (size_t)min(t0 + i, T - 1) * K + k);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        uint32_t o[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int i = 0; i < 16; ++i) o[i >> 2] |= (t0 + i < T ? (w[i] >> (8 * j)) & 0xFFu : 0u) << (8 * (i & 3));
        *reinterpret_cast<uint4*>(qT + (size_t)(k + j) * Tp + t0) = make_uint4(o[0], o[1], o[2], o[3]);
        int z = -max(t0 + 16 - T, 0);                // (not the padding)
#pragma unroll
        for (int i = 0; i < 4; ++i) z += __builtin_popcount(~(((o[i] & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | o[i] | 0x7F7F7F7Fu));
        atomicAdd(&zero_codes[4 * lane + j], z);
      }
    }
    __syncthreads();
    const int kk = k0 + threadIdx.x;
    if (kk < K && zero_codes[threadIdx.x] > 0) atomicAdd(counts + 2 * N + kk, zero_codes[threadIdx.x]);
    return;
  }
  const int n = blockIdx.x * 64 + lane;
  if (n >= N) return;
  const int e = cexp[n];
  const bool ok = e != PQ_FIXED_NOT_FINITE;
  const double s = ok ? pow2(min(54 - e, 1023)) : 0.0;
  const int tend = min(Tp, (int)(blockIdx.y + 1) * COLT);
  int small = 0, zero = 0;
  for (int t0 = blockIdx.y * COLT + wv * 16; t0 < tend; t0 += 64) {
    float v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = dY[(size_t)min(t0 + i, T - 1) * N + n];
    uint32_t o[4][ND];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      uint64_t w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = t0 + 4 * h + i;
        const double x = (double)v[4 * h + i] * recip(gamma[min(t, T - 1)]) * s;
        w[i] = ok && t < T ? digits(x) : 0;
        const bool is0 = t < T && v[4 * h + i] == 0.0f;
        zero += is0 ? 1 : 0;
        small += t < T && !is0 && fabs(x) < (double)(1ull << SMALL) ? 1 : 0;
      }
      planes_of(w, o[h]);
    }
#pragma unroll
    for (int d = 0; d < ND; ++d)
      *reinterpret_cast<uint4*>(D + ((size_t)d * N + n) * Tp + t0) = make_uint4(o[0][d], o[1][d], o[2][d], o[3][d]);
  }
  if (small > 0) atomicAdd(counts + n, small);       // (rare on both counts)
  if (zero > 0) atomicAdd(counts + N + n, zero);
}

}  // namespace

int pq_fixed_max_rows(int T) { return (T + ROWS - 1) / ROWS; }

int pq_launch_fixed_split(const float* dY, const float* gamma, const int8_t* q, int T, int Tp, int N, int K, int8_t* Drow, int* rexp, int8_t* Dcol,
                          int* cexp, int8_t* qT, uint32_t* colmax, int* counts, hipStream_t s) {
  pq_prof_scope prof(PQP_QUANT, s);
  fixed_rows_kernel<<<pq_fixed_max_rows(T), 512, 0, s>>>(dY, gamma, T, N, Drow, rexp, colmax, counts, 2 * N + K);
  PQ_CHECK_LAUNCH("fixed_rows_kernel");
  const int nblk = (N + 63) / 64;
  fixed_exps_kernel<<<nblk, 1024, 0, s>>>(colmax, pq_fixed_max_rows(T), N, cexp);
  PQ_CHECK_LAUNCH("fixed_exps_kernel");
  fixed_cols_kernel<<<dim3(nblk + (K + 255) / 256, (Tp + COLT - 1) / COLT), 256, 0, s>>>(dY, gamma, q, T, Tp, N, K, cexp, Dcol, qT, counts, nblk);
  PQ_CHECK_LAUNCH("fixed_cols_kernel");
  return PQ_OK;
}
