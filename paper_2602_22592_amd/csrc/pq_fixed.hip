// fp32 I/O, large products: the two big contractions of the backward, dX = dY S and dW = (dY / gamma)^T q, as exact integer
// products on the int8 matrix pipe.
//
// One operand of each is already small integers (signs, codes), so only dY has to be cut up: a row of the left operand (a
// token of dY, or an output channel over the tokens) is written as fixed-point numbers of 55 bits relative to its largest
// element, X = rint(x 2^(54 - E)), max |x| < 2^E, and those as seven signed digits of base 256, each in a byte (the
// splitting of operands into slices whose products are exact: Ozaki, Ogita, Oishi, Rump, "Error-free transformations of matrix
// multiplication", 2012).  Seven int8 products with int32 sums are exact; their sum sum_d 256^d acc_d 2^(E - 54) is formed in fp64 by
// the kernel that multiplies them, and the fp64 engine (pq_ref.hip, the SUM forms) adds what belongs to it and rounds.  What is lost is the rounding of an element to 2^(E - 55).  In dX every element of a row enters every
// sum, and the additions behind the largest one round as much in fp64.  In dW a token whose code is zero stays out of a sum, and the
// largest element may be such a token's.  The column pass therefore counts the small elements, below 2^(E - 17), the zero ones and,
// per channel, the zero codes; a sum is taken from the digits only if, with l = tokens - small - zero ones and z the zero codes,
//     8 max(l - z, 0) >= min(small, tokens - z):
// at least l - z larger elements enter it then and at most eight times as many small ones, so that it is off by at most 2^-28 of
// sum |x q|, a sixteenth of the rounding to fp32.  A 32x32 tile with another sum in it
// is formed as the fp64 product it stands for.  One token 1e9 / 1e12 / 1e16 times the others: relative error of the sums that its zero
// codes leave out 3.2e-8 / 1.9e-5 / 0.2 from the digits, 2.6e-8 now.  Backward of 2048 tokens 2048x2048 (us): 166 with normal data; 154 to
// 165 with 95 % zero codes, half of the tokens masked, token scales of e^+-6 or elements of e^+-10; 476 with one token 1e6 times the others
// (all tiles fp64).
// What it is for: the fp64 matrix rate is 78.6 TFLOP/s, the int8 one 5 POP/s nominal and 2 on real data, so seven products cost a
// quarter of one fp64 product.  2048 tokens, 2048x2048, r = 128, whole step (us): 718 with every product in fp64, 380 with the digits' int32 sums
// added up from memory, 326 with the sums formed where they are multiplied; the passes below 13, 5 and 16, two of them over dY, 4 bytes read
// and 7 written per element.
// Infinities and NaN have no fixed-point form: their rows get no digits and are marked, and the SUM forms compute a 32x32 tile that
// a marked row reaches as the fp64 product it stands for.  Step of 2048 tokens 2048x2048 without a branch (us): finite 206; one NaN in dY 363; an infinity in X, which marks every
// row of dW, 515 (one element after the other: 1115 and 5368; fp64 products alone 594).
#include <string.h>
#include <type_traits>
#include "pq_epilogue.h"

namespace {

constexpr int ND = PQ_FIXED_DIGITS;
constexpr int COLT = 128;                            // tokens per workgroup of the column pass
constexpr int SMALL = 37;                            // digits below 2^37: elements below 2^(E - 17)
constexpr int ROWS = 8;                              // rows of dY per workgroup of the row pass, four to a half of it
constexpr int FXM = PQ_FIXED_M, FXN = PQ_FIXED_N;    // the products' tiles

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

// What the products read lies in memory as the tiles that they stream: panels of FXM rows (digits) or FXN rows (signs, codes), stages of 64
// contraction indices, and in a stage [digit][row][64 B] with the row's 16-byte chunks swizzled, so that every direct load is 1 KB of
// consecutive memory and lands where the operand reads want it.  (As plain rows the loads took 64 bytes of sixteen rows: 103 us for the
// stream of 2048 tokens 2048x2048 alone; and the column pass below stored 16-byte pieces a row apart.)  Bytes of chunk c of row r:
__device__ __forceinline__ int tile_off(int r, int c) { return r * 64 + (((c ^ (r >> 1) ^ (r >> 3)) & 3) << 4); }

// Rows of dY: digits (panels of 64 tokens) and exponents [T]; colmax [ceil(T / ROWS)][N]: the largest |dY / gamma| of the workgroup's rows, as
// the upper half of the double.  counts: cleared for the column pass.
__global__ __launch_bounds__(512) void fixed_rows_kernel(const float* __restrict__ dY, const float* __restrict__ gamma, int T, int N,
                                                         int8_t* __restrict__ D, int* __restrict__ rexp, uint32_t* __restrict__ colmax,
                                                         int* __restrict__ counts, int ncounts, const uint16_t* __restrict__ bits,
                                                         int8_t* __restrict__ signs, int K, int nrow) {
  const int nk = (N + 63) >> 6;                      // stages of a contraction over the columns
  if ((int)blockIdx.x >= nrow) {                     // uniform: the packed signs [K][N] as bytes, a chunk per thread and turn, zeros behind a row's end
    const size_t total = (size_t)K * nk * 4;
    for (size_t i = (size_t)((int)blockIdx.x - nrow) * 512 + threadIdx.x; i < total; i += (size_t)((int)gridDim.x - nrow) * 512) {
      const int k = (int)(i / (unsigned)(nk * 4)), ch = (int)(i - (size_t)k * (nk * 4));
      const i32x4_t o = ch * 16 < N ? pq_bits_to_i8(bits[(size_t)k * (N >> 4) + ch]) : i32x4_t{0, 0, 0, 0};
      *reinterpret_cast<i32x4_t*>(signs + ((size_t)(k / FXN) * nk + (ch >> 2)) * (FXN * 64) + tile_off(k % FXN, ch & 3)) = o;
    }
    return;
  }
  for (int i = blockIdx.x * 512 + threadIdx.x; i < ncounts; i += nrow * 512) counts[i] = 0;
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
      for (int d = 0; d < ND; ++d)
        *reinterpret_cast<uint32_t*>(D + (((size_t)((t0 + r) / FXM) * nk + (c >> 6)) * ND + d) * (FXM * 64) + tile_off((t0 + r) % FXM, (c >> 4) & 3) + (c & 15)) = o[d];
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

// Columns of dY / gamma over the tokens: digits (panels of 64 columns); and q transposed (panels of 128 channels).  Tp: T rounded up to
// whole stages, the rest zero.  counts: small elements [N], zero ones [N], zero codes [K].  Workgroups (column block, token block of COLT): N / 64 of digits, then K / 256 of codes.
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
        *reinterpret_cast<uint4*>(qT + ((size_t)((k + j) / FXN) * (Tp >> 6) + (t0 >> 6)) * (FXN * 64) + tile_off((k + j) % FXN, (t0 >> 4) & 3)) =
            make_uint4(o[0], o[1], o[2], o[3]);
        int z = -min(max(t0 + 16 - T, 0), 16);       // (not the padding)
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
      *reinterpret_cast<uint4*>(D + (((size_t)blockIdx.x * (Tp >> 6) + (t0 >> 6)) * ND + d) * (FXM * 64) + tile_off(lane, (t0 >> 4) & 3)) =
          make_uint4(o[0][d], o[1][d], o[2][d], o[3][d]);
  }
  if (small > 0) atomicAdd(counts + n, small);       // (rare on both counts)
  if (zero > 0) atomicAdd(counts + N + n, zero);
}

// ---------------------------------------------------------------------------------------------
// The sums of the digit products: S[m][n] = sum_d 256^d (sum_k A_d(m,k) B(n,k)) 2^(E_m - 54) (A_d: the d-th digits of dY's rows or
// columns; B: signs or transposed codes).
// ---------------------------------------------------------------------------------------------
// A wavefront multiplies 32 rows of all seven digits with 64 columns: fourteen 32x32 blocks of int32 sums (224 AGPRs, one wavefront
// per SIMD), which meet in fp64 in its own registers.  As one product of 7 M rows with its int32 planes in memory the same work wrote and
// read 56 bytes per output and fetched the operand B once per digit; here a B operand read from LDS serves seven MFMAs (nine operand
// reads to fourteen MFMAs) and an output leaves as 8 bytes.  A workgroup is 64x128 outputs on four wavefronts (2 x 2); a stage is 64
// contraction indices (36 KB), the ring has four.  The order of a stage is fixed, as in the weight-gradient products: behind the MFMAs of
// the first half go the operand reads of the second, then the barrier, then the direct loads of the stage three ahead; behind those of
// the second half the operand reads of the next stage, which that barrier has let in.
// One workgroup per CU walks over tiles, and its loads run on into the next tile: the conversion and the stores of a tile (6 us where a
// tile was a workgroup, against 19 of MFMAs) have the next one's first three stages under way.
constexpr int FX_A = ND * FXM * 64, FX_STAGE = FX_A + FXN * 64, FX_OUT = 4096;   // bytes of a stage, and of a wavefront's share of the output's patch

struct fixed_product {
  const int8_t* A;      // [M / 64][nkt][ND][64][64 B]
  const int8_t* B;      // [N / 128][nkt][128][64 B]
  const int* exps;      // [M]
  double* S;            // [M][N]
  int M, N, nkt, nbn;
};

#define FX_MFMA(acc, a, b) asm volatile("v_mfma_i32_32x32x32_i8 %0, %2, %1, %0" : "+a"(acc) : "v"(a), "v"(b))
#define FX_MFMA0(acc, a, b) asm volatile("v_mfma_i32_32x32x32_i8 %0, %2, %1, 0" : "=a"(acc) : "v"(a), "v"(b))
#define FX_READ(dst, addr, off) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(off) : "memory")
struct fixed_frags {
  i32x4_t q[ND + 2];    // the digits' operands, then the two of B
  __device__ __forceinline__ void wait_all() {
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(q[0]), "+v"(q[1]), "+v"(q[2]), "+v"(q[3]), "+v"(q[4]), "+v"(q[5]), "+v"(q[6]), "+v"(q[7]), "+v"(q[8]));
  }
};

__global__ __launch_bounds__(256, 1) void fixed_gemm_kernel(fixed_product p0, fixed_product p1, int tiles0, int tiles) {
#if defined(__HIP_DEVICE_COMPILE__)
  static_assert(ND == 7 && FXM == 64 && FXN == 128, "nine load instructions per wavefront and stage");
  constexpr int IPS = FX_STAGE / 4096;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[4 * FX_STAGE + 4 * FX_OUT];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wv >> 1, wn = wv & 1;
  // tiles of this workgroup: every gridDim.x-th; of each round an XCD (workgroups c, c + 8, ..) takes consecutive ones
  const int per = (int)gridDim.x >> 3;
  const int tile_first = ((int)gridDim.x & 7) == 0 ? ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3) : (int)blockIdx.x;
  if (tile_first >= tiles) return;                              // uniform

  // ---- the load stream: stage after stage, tile after tile ----
  const int8_t *la, *lb;                                        // of the next stage to request
  int lt = tile_first, lk = 0, lnkt = 0;
  auto load_tile = [&] {
    const bool sec = lt >= tiles0;
    const int t = sec ? lt - tiles0 : lt, nbn = sec ? p1.nbn : p0.nbn;
    lnkt = sec ? p1.nkt : p0.nkt;
    la = (sec ? p1.A : p0.A) + (size_t)(t / nbn) * lnkt * FX_A;
    lb = (sec ? p1.B : p0.B) + (size_t)(t % nbn) * lnkt * (FXN * 64);
  };
  load_tile();
  auto issue1 = [&](int slot, int i) {
    const int qi = wv * IPS + i;                                // 1 KB block of the stage
    const int8_t* g = (qi < ND * 4 ? la + qi * 1024 : lb + (qi - ND * 4) * 1024) + lane * 16;
    __builtin_amdgcn_global_load_lds(g, PQ_LDS_PTR(smem + slot * FX_STAGE + qi * 1024), 16, 0, 0);
  };
  auto advance = [&] {                                          // past the last stage: it again, into a slot nobody reads
    if (++lk < lnkt) {
      la += FX_A;
      lb += FXN * 64;
    } else if (lt + (int)gridDim.x < tiles) {
      lt += (int)gridDim.x;
      lk = 0;
      load_tile();
    }
  };
#pragma unroll
  for (int u = 0; u < 3; ++u) {
#pragma unroll
    for (int i = 0; i < IPS; ++i) issue1(u, i);
    advance();
  }

  // operand reads (slot 0): lane l takes row l & 31, chunk 2 ks + (l >> 5); 32 rows further the swizzle is the same
  const uint32_t lds0 = (uint32_t)(size_t)smem;
  uint32_t adA[2], adB[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int o = tile_off(lane & 31, 2 * ks + (lane >> 5));
    adA[ks] = lds0 + wm * 2048 + o;
    adB[ks] = lds0 + FX_A + wn * 4096 + o;
  }
  fixed_frags F0, F1;
  auto rd = [&](fixed_frags& F, int n, uint32_t so, int ks) {   // B first: every MFMA needs one of them
    if (n < 2) {
      const uint32_t pb = adB[ks] + so;
      if (n == 0) FX_READ(F.q[ND], pb, 0);
      else FX_READ(F.q[ND + 1], pb, 2048);
    } else {
      const uint32_t pa = adA[ks] + so;
      switch (n - 2) {                                          // (constant after unrolling)
        case 0: FX_READ(F.q[0], pa, 0); break;
        case 1: FX_READ(F.q[1], pa, 4096); break;
        case 2: FX_READ(F.q[2], pa, 8192); break;
        case 3: FX_READ(F.q[3], pa, 12288); break;
        case 4: FX_READ(F.q[4], pa, 16384); break;
        case 5: FX_READ(F.q[5], pa, 20480); break;
        default: FX_READ(F.q[6], pa, 24576);
      }
    }
  };
  i32x16_t acc[ND][2];
  auto mf = [&acc](const fixed_frags& X, int n, auto first_c) {    // an operand of A stays for two MFMAs
    const int d = n >> 1, j = (n & 1) ^ (d & 1);
    if constexpr (decltype(first_c)::value) FX_MFMA0(acc[d][j], X.q[d], X.q[ND + j]);
    else FX_MFMA(acc[d][j], X.q[d], X.q[ND + j]);
  };
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  asm volatile("s_barrier" ::: "memory");
#pragma unroll
  for (int n = 0; n < ND + 2; ++n) rd(F0, n, 0u, 0);

  int slot = 0;
  for (int tile = tile_first; tile < tiles; tile += (int)gridDim.x) {
    const bool sec = tile >= tiles0;                            // uniform
    const int nkt = sec ? p1.nkt : p0.nkt;
    for (int kt = 0; kt < nkt; ++kt) {
      const uint32_t so = (uint32_t)slot * FX_STAGE, sn = (uint32_t)((slot + 1) & 3) * FX_STAGE;
      const int sl = (slot + 3) & 3;
      F0.wait_all();
      auto half = [&](auto first_c) {
#pragma unroll
        for (int n = 0; n < ND; ++n) {
          mf(F0, n, first_c);
          rd(F1, n, so, 1);
          if (n < 2) rd(F1, n + ND, so, 1);
        }
        // The wavefront's own loads of the next stage have landed.  (At a tile's start there are three stages that the end of the
        // tile before, or the start, has waited for, and stores behind them that nothing here need wait for.)
        if constexpr (!decltype(first_c)::value)
          if (kt > 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(IPS) : "memory");
        asm volatile("s_barrier" ::: "memory");                 // everybody's have; nobody reads the stage before this one any more
#pragma unroll
        for (int n = ND; n < 2 * ND; ++n) {
          mf(F0, n, first_c);
          issue1(sl, n - ND);
          if (n < ND + 2) issue1(sl, n);
        }
      };
      if (kt == 0) half(std::true_type{});
      else half(std::false_type{});
      advance();
      F1.wait_all();
#pragma unroll
      for (int n = 0; n < 2 * ND; ++n) {
        mf(F1, n, std::false_type{});
        if (n < ND + 2) rd(F0, n, sn, 0);                       // past the last stage: a slot nobody uses
      }
      slot = (slot + 1) & 3;
    }
    // The operand reads of the next tile have landed before the compiler has registers to place: it takes their outputs as written.
    F0.wait_all();
    // (an asm MFMA's registers may be read when the matrix pipe has written them: the compiler does not know)
    asm volatile("s_nop 15\n\ts_nop 3" ::: "memory");
#pragma unroll
    for (int d = 0; d < ND; ++d)
#pragma unroll
      for (int j = 0; j < 2; ++j) asm volatile("" : "+a"(acc[d][j]));

    // In a block lane l holds row l & 31, register v column 8 (v >> 2) + 4 (l >> 5) + (v & 3).  Sixteen columns at a time pass through
    // the wavefront's patch, [32 rows][128 B], and leave as whole lines.
    const fixed_product& p = sec ? p1 : p0;
    const int t = sec ? tile - tiles0 : tile;
    const int m0 = t / p.nbn * FXM + wm * 32, n0 = t % p.nbn * FXN + wn * 64;
    const int row = lane & 31;
    const int e = p.exps[min(m0 + row, p.M - 1)];
    const double sc = e == PQ_FIXED_NOT_FINITE ? 0.0 : ldexp(1.0, e - 54);
    unsigned char* const mine = smem + 4 * FX_STAGE + wv * FX_OUT;
#pragma unroll
    for (int c = 0; c < 4; ++c) {                               // columns 16 c .. 16 c + 15
      double2 o[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int j = c >> 1, v = 8 * (c & 1) + 2 * x;
        double s[2] = {0.0, 0.0};
#pragma unroll
        for (int d = ND - 1; d >= 0; --d)
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int a = acc[d][j][v + u];
            s[u] = __builtin_fma(s[u], 256.0, (double)a);
          }
        o[x] = make_double2(s[0] * sc, s[1] * sc);
      }
      if (c == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the next tile's stages, ahead of the stores
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int ch = (x >> 1) * 4 + (lane >> 5) * 2 + (x & 1);     // 16-byte chunk of the row's 128 bytes
        const uint32_t ad = (uint32_t)(size_t)(mine + row * 128 + ((ch ^ (row & 7)) << 4));
        const i32x4_t w = __builtin_bit_cast(i32x4_t, o[x]);
        // (asm with two wait states behind it: see the staged epilogue of mfma_gemm_kernel)
        asm volatile("ds_write_b128 %0, %1\n\ts_nop 1" ::"v"(ad), "v"(w) : "memory");
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int r = it * 8 + (lane >> 3), ch = lane & 7;
        const double2 w = *reinterpret_cast<const double2*>(mine + r * 128 + ((ch ^ (r & 7)) << 4));
        const int m = m0 + r, n = n0 + c * 16 + ch * 2;
        if (m < p.M && n < p.N) *reinterpret_cast<double2*>(p.S + (size_t)m * p.N + n) = w;   // (N is even)
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#endif
}

}  // namespace

int pq_fixed_max_rows(int T) { return (T + ROWS - 1) / ROWS; }

int pq_launch_fixed_split(const float* dY, const float* gamma, const int8_t* q, int T, int N, int K, int8_t* Drow, int* rexp, int8_t* Dcol,
                          int* cexp, int8_t* qT, uint32_t* colmax, int* counts, const uint32_t* Pt, int8_t* signs, hipStream_t s) {
  pq_prof_scope prof(PQP_QUANT, s);
  const int nrow = pq_fixed_max_rows(T), Tp = (T + 63) / 64 * 64;
  const size_t chunks = (size_t)K * ((N + 63) / 64) * 4;
  const int nsign = (int)((chunks + 2047) / 2048 < 1024 ? (chunks + 2047) / 2048 : 1024);
  fixed_rows_kernel<<<nrow + nsign, 512, 0, s>>>(dY, gamma, T, N, Drow, rexp, colmax, counts, 2 * N + K, (const uint16_t*)Pt, signs, K, nrow);
  PQ_CHECK_LAUNCH("fixed_rows_kernel");
  const int nblk = (N + 63) / 64;
  fixed_exps_kernel<<<nblk, 1024, 0, s>>>(colmax, pq_fixed_max_rows(T), N, cexp);
  PQ_CHECK_LAUNCH("fixed_exps_kernel");
  fixed_cols_kernel<<<dim3(nblk + (K + 255) / 256, (Tp + COLT - 1) / COLT), 256, 0, s>>>(dY, gamma, q, T, Tp, N, K, cexp, Dcol, qT, counts, nblk);
  PQ_CHECK_LAUNCH("fixed_cols_kernel");
  return PQ_OK;
}

int pq_launch_fixed_products(const int8_t* Drow, const int* rexp, const int8_t* signs, double* SX, const int8_t* Dcol, const int* cexp, const int8_t* qT,
                             double* SW, int T, int N, int K, hipStream_t s) {
  if (T <= 0 || N <= 0 || N % 32 != 0 || K <= 0 || K % 32 != 0) return pq_set_error(PQ_ERR_SHAPE, "digit products: T=%d d_in=%d d_out=%d", T, K, N);
  pq_prof_scope prof(PQP_GEMM_DX, s);               // (dW's products too)
  const int nbn = (K + FXN - 1) / FXN;
  const fixed_product x{Drow, signs, rexp, SX, T, K, (N + 63) / 64, nbn}, w{Dcol, qT, cexp, SW, N, K, (T + 63) / 64, nbn};
  const int tx = (T + FXM - 1) / FXM * nbn, tw = (N + FXM - 1) / FXM * nbn, tiles = tx + tw;
  const bool w_first = T >= N;                       // the longer contraction first
  fixed_gemm_kernel<<<tiles < 256 ? tiles : 256, 256, 0, s>>>(w_first ? w : x, w_first ? x : w, w_first ? tw : tx, tiles);
  PQ_CHECK_LAUNCH("fixed_gemm_kernel");
  return PQ_OK;
}
