// C = A B on SM-packed operands, exact, written densely into scratch with the
// exact range of C (the max-reduction pass that fixes C's width).  Products
// run on the matrix cores (gemm_limb.hpp) over operands decoded here; the
// generic path below takes what that path cannot (K of 2^17 or more, and a
// scratch that holds no more than C) and short sums (matmul_fast_bytes).
//
// Generic path (any widths): 64x64 output tiles per 256-lane block, K in
// chunks of 32.  Each chunk of A (64x32) and B (32x64) is decoded from the
// packed streams straight into LDS; every lane then accumulates a 4x4
// micro-tile in int64.  The overflow rule checked on the host (K * max|A| *
// max|B| < 2^63) makes every partial sum exact.
#include "ccm_internal.hpp"
#include "gemm_limb.hpp"
#include "mv_tile.hpp"
#include "group_codec.hpp"

namespace ccm {
namespace {

constexpr int kTM = 64, kTN = 64, kTK = 32, kThreads = 256;

template <typename ET, typename OT>
__global__ __launch_bounds__(kThreads) void k_gemm_generic(
    const uint32_t *__restrict__ aw, int abits, int asgn, const uint32_t *__restrict__ bw,
    int bbits, int bsgn, int64_t M, int64_t K, int64_t N, OT *__restrict__ C, RangeSink sink) {
  __shared__ ET As[kTK][kTM + 1];  // As[k][m]
  __shared__ ET Bs[kTK][kTN + 1];  // Bs[k][n]
  const int64_t gx = (N + kTN - 1) / kTN;
  const int64_t m0 = blockIdx.x / gx * kTM, n0 = blockIdx.x % gx * kTN;
  const int tid = threadIdx.x;
  const int tm = (tid / 16) * 4, tn = (tid % 16) * 4;
  int64_t acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0;

  for (int64_t k0 = 0; k0 < K; k0 += kTK) {
    for (int q = tid; q < kTM * kTK; q += kThreads) {
      const int mm = q / kTK, kk = q % kTK;
      const int64_t m = m0 + mm, k = k0 + kk;
      As[kk][mm] = (m < M && k < K) ? (ET)value_at(aw, (uint64_t)(m * K + k), abits, asgn) : ET(0);
    }
    for (int q = tid; q < kTK * kTN; q += kThreads) {
      const int kk = q / kTN, nn = q % kTN;
      const int64_t k = k0 + kk, n = n0 + nn;
      Bs[kk][nn] = (k < K && n < N) ? (ET)value_at(bw, (uint64_t)(k * N + n), bbits, bsgn) : ET(0);
    }
    __syncthreads();
#pragma unroll 4
    for (int kk = 0; kk < kTK; ++kk) {
      ET a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[kk][tm + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Bs[kk][tn + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] += (int64_t)a[i] * (int64_t)b[j];
    }
    __syncthreads();
  }

  int64_t lo = INT64_MAX, hi = INT64_MIN;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t m = m0 + tm + i;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t n = n0 + tn + j;
      if (m < M && n < N) {
        const int64_t v = acc[i][j];
        C[m * N + n] = (OT)v;
        lo = v < lo ? v : lo;
        hi = v > hi ? v : hi;
      }
    }
  }
  block_range_commit(lo, hi, 0, sink);
}

template <typename ET>
hipError_t launch_generic(const uint32_t *aw, int abits, int asgn, const uint32_t *bw,
                          int bbits, int bsgn, int64_t M, int64_t K, int64_t N, int out32,
                          void *scratch, RangeSink sink, hipStream_t s) {
  // in one dimension: a second one ends at 65535 blocks, 4.2 million rows
  const uint64_t tiles = (uint64_t)((N + kTN - 1) / kTN) * (uint64_t)((M + kTM - 1) / kTM);
  if (!launch_fits(tiles, kThreads)) return hipErrorInvalidValue;
  const unsigned grid = (unsigned)tiles;
  if (out32)
    k_gemm_generic<ET, int32_t><<<grid, kThreads, 0, s>>>(aw, abits, asgn, bw, bbits, bsgn, M,
                                                          K, N, (int32_t *)scratch, sink);
  else
    k_gemm_generic<ET, int64_t><<<grid, kThreads, 0, s>>>(aw, abits, asgn, bw, bbits, bsgn, M,
                                                          K, N, (int64_t *)scratch, sink);
  return hipGetLastError();
}

// ---- matrix-core path: the operands' digits --------------------------------
//
// Both operands are first decoded once into base-256 digits (gemm_limb.hpp)
// with K contiguous and zero-padded to a multiple of the K step: A as M rows,
// B transposed as N rows (B^T, the paper's other unravel order).  Decoding
// inside the GEMM's K loop would redo it for every output tile (N/256 times
// per A element) and read the packed rows one lane per row, which the memory
// pipeline serves one cache line per lane; decoded once, the tiles stream with
// coalesced 16-byte copies.  Both decoding kernels are bound by HBM: packed
// bytes in, L bytes an element out.

using limb::Limbs;

__host__ __device__ inline int64_t padded_k(int64_t K) {
  return (K + limb::kBK - 1) / limb::kBK * limb::kBK;
}

// Rows an operand of L limbs takes per limb: its own, or for several limbs
// whole groups of 32.
__host__ __device__ inline int64_t limb_rows(int64_t rows, int L) {
  return L == 1 ? rows : (rows + 31) / 32 * 32;
}

// Stacked row of (row, limb i) counted from the operand's first.
__device__ __forceinline__ int64_t stacked_row(int64_t row, int i, int64_t rows, Limbs L) {
  if (L.n == 1) return row;
  const int c0 = i / L.chunk * L.chunk;
  const int lc = L.n - c0 < L.chunk ? L.n - c0 : L.chunk;
  return c0 * limb_rows(rows, L.n) + ((row >> 5) * lc + (i - c0)) * 32 + (row & 31);
}

// The digits of a group of 32 fields of B <= 32 bits starting at stream bit
// `bit`, `lim` of them real (the others 0): o[i][q] = digit i of fields
// 4q..4q+3.
template <int B>
__device__ __forceinline__ void group_digits(const uint32_t *__restrict__ w, uint64_t cap,
                                             uint64_t bit, int sgn, int lim,
                                             uint32_t (&o)[(B + 7) / 8][8]) {
  constexpr int L = (B + 7) / 8;
  const uint64_t w0 = bit >> 5;
  const int sh = (int)(bit & 31u);
  uint32_t ww[B + 1];
#pragma unroll
  for (int q = 0; q <= B; ++q) ww[q] = w[w0 + q < cap ? w0 + q : cap - 1];
#pragma unroll
  for (int q = 0; q < B; ++q) ww[q] = __builtin_amdgcn_alignbit(ww[q + 1], ww[q], sh);
  limb::words_digits<B>(ww, sgn, o);
  if (lim < 32) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int left = lim - 4 * q;
      const uint32_t m = left >= 4 ? ~0u : left <= 0 ? 0u : (1u << (8 * left)) - 1u;
#pragma unroll
      for (int i = 0; i < L; ++i) o[i][q] &= m;
    }
  }
}

using limb::sum4;

// The block's sum of one value per thread, in thread 0.
__device__ __forceinline__ int64_t block_sum(int64_t v) {
  __shared__ int64_t s_part[4];
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = v;
  __syncthreads();
  int64_t t = 0;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += s_part[i];
  return t;
}

// The column addends (null: none) start at zero; the kernel that adds to them
// runs after this one.
__device__ __forceinline__ void zero_cadd(int64_t *__restrict__ cadd, int64_t N) {
  if (!cadd) return;
  for (int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x; n < N; n += (int64_t)gridDim.x * 256)
    cadd[n] = 0;
}

// Digits of A: one block per row, lane j takes columns 32j..32j+31 (one
// group's worth of fields, re-aligned with a funnel shift when the row starts
// inside a word).  radd (may be null): radd[row] = beta times the sum of the
// row's values less their offsets.
template <int B>
__global__ __launch_bounds__(256) void k_digit_rows(const uint32_t *__restrict__ w, uint64_t cap,
                                                    int sgn, int64_t M, int64_t K, int64_t ldk,
                                                    Limbs L, int8_t *__restrict__ out,
                                                    uint64_t beta, int64_t *__restrict__ radd,
                                                    int64_t *__restrict__ cadd, int64_t N) {
  constexpr int LB = (B + 7) / 8;
  const int64_t row = blockIdx.x;
  zero_cadd(cadd, N);
  uint64_t sum = 0;
  for (int64_t c = 32 * (int64_t)threadIdx.x; c < ldk; c += 32 * 256) {
    uint32_t o[LB][8];
    if (c < K) {
      group_digits<B>(w, cap, ((uint64_t)row * (uint64_t)K + (uint64_t)c) * B, sgn,
                      K - c < 32 ? (int)(K - c) : 32, o);
    } else {
#pragma unroll
      for (int i = 0; i < LB; ++i)
#pragma unroll
        for (int q = 0; q < 8; ++q) o[i][q] = 0;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      uint4 *d = reinterpret_cast<uint4 *>(out + stacked_row(row, i, M, L) * ldk + c);
      d[0] = make_uint4(o[i][0], o[i][1], o[i][2], o[i][3]);
      d[1] = make_uint4(o[i][4], o[i][5], o[i][6], o[i][7]);
      if (radd) {
        int t = 0;
#pragma unroll
        for (int q = 0; q < 8; ++q) t = sum4(o[i][q], t);
        sum += (uint64_t)(int64_t)t << (8 * i);
      }
    }
  }
  if (radd) {
    const int64_t t = block_sum((int64_t)sum);
    if (threadIdx.x == 0) radd[row] = (int64_t)(beta * (uint64_t)t);
  }
}

// As k_digit_rows for fields of 33..64 bits: a lane takes four columns at a
// time, its fields read one by one (the products outnumber them by far).
__global__ __launch_bounds__(256) void k_digit_rows_wide(const uint32_t *__restrict__ w, int bits,
                                                         int sgn, int64_t M, int64_t K,
                                                         int64_t ldk, Limbs L,
                                                         int8_t *__restrict__ out, uint64_t beta,
                                                         int64_t *__restrict__ radd,
                                                         int64_t *__restrict__ cadd, int64_t N) {
  const int64_t row = blockIdx.x;
  zero_cadd(cadd, N);
  uint64_t sum = 0;
  for (int64_t c = 4 * (int64_t)threadIdx.x; c < ldk; c += 4 * 256) {
    uint64_t v[4];
    uint32_t live = 0;
    for (int q = 0; q < 4; ++q) {
      const bool in = c + q < K;
      v[q] = in ? (uint64_t)value_at(w, (uint64_t)(row * K + c + q), bits, sgn) : 0;
      live |= in ? 0xffu << (8 * q) : 0u;
    }
    for (int i = 0; i < L.n; ++i) {
      uint32_t o = 0;
      for (int q = 0; q < 4; ++q) o |= (uint32_t)((v[q] >> (8 * i)) & 0xff) << (8 * q);
      o = (o ^ limb::digit_flip(bits, sgn, i, L.n)) & live;
      *reinterpret_cast<uint32_t *>(out + stacked_row(row, i, M, L) * ldk + c) = o;
      sum += (uint64_t)(int64_t)sum4(o, 0) << (8 * i);
    }
  }
  if (radd) {
    const int64_t t = block_sum((int64_t)sum);
    if (threadIdx.x == 0) radd[row] = (int64_t)(beta * (uint64_t)t);
  }
}

// cadd[n] += alpha (sum + live beta), from the sums of the four lanes of n
__device__ __forceinline__ void commit_col(uint64_t sum, int kq, int64_t n, int64_t N, int64_t live,
                                           uint64_t alpha, uint64_t beta,
                                           int64_t *__restrict__ cadd) {
  sum += (uint64_t)__shfl_xor((long long)sum, 1, 64);
  sum += (uint64_t)__shfl_xor((long long)sum, 2, 64);
  if (kq == 0 && n < N)
    atomicAdd((unsigned long long *)&cadd[n],
              (unsigned long long)(alpha * (sum + (uint64_t)live * beta)));
}

// Digits of B^T (out row n holds column n of B), through an LDS tile per limb of
// 128 k x TN n (256, 128 or 64 by the number of limbs, 33 KB in all):
//   * each lane decodes groups (32 consecutive n of one row k of B, read as the
//     group's words): at 4 bits a row's 256 fields are a whole line, where 64 of
//     them left each line to four blocks, on four XCDs;
//   * a lane turns 4 n x 32 k of a limb around, four words at a time (eight byte
//     permutes instead of sixteen byte reads), and writes two 16-byte chunks per
//     n: lane kq of four takes the 16 k from 16 kq and from 64 + 16 kq, whose rows
//     then lie 16 banks apart (the four lanes and their 16 n-quads fill the 64).
// cadd (may be null, else zero before the launch): cadd[n] += alpha times the sum
// of column n's values.  tiles > 0 (one digit): out in chunk tiles for `tiles`
// blocks of 16 columns instead of rows (gemm_narrow.hpp).
// Bound by memory: packed words in, L bytes an element out.  8192 x 8192 at 4
// bits: 27 us, 42 with tiles of 64 n read back by bytes.
constexpr int kCtK = 128;
// n of a tile; `wide`: as many as the LDS budget gives.
constexpr int ct_cols(int limbs, bool wide) {
  return !wide || limbs > 2 ? 64 : limbs == 2 ? 128 : 256;
}

template <int B, int TN>
__global__ __launch_bounds__(256) void k_digit_cols(const uint32_t *__restrict__ w, uint64_t cap,
                                                    int sgn, int64_t K, int64_t N, int64_t ldk,
                                                    Limbs L, int8_t *__restrict__ out,
                                                    uint64_t alpha, uint64_t beta,
                                                    int64_t *__restrict__ cadd, int tiles) {
  constexpr int LB = (B + 7) / 8, kPitch = TN / 4 + 1;  // words
  __shared__ uint32_t tile[LB][kCtK * kPitch];
  const int64_t nb = (int64_t)blockIdx.x * TN, kb = (int64_t)blockIdx.y * kCtK;
  constexpr int G = TN / 32;
#pragma unroll 1
  for (int r = 0; r < kCtK * G / 256; ++r) {
    const int t = r * 256 + threadIdx.x;
    const int kl = t / G, g = t % G;
    const int64_t k = kb + kl, n0 = nb + 32 * g;
    uint32_t o[LB][8];
    if (k < K && n0 < N) {
      group_digits<B>(w, cap, ((uint64_t)k * (uint64_t)N + (uint64_t)n0) * B, sgn,
                      N - n0 < 32 ? (int)(N - n0) : 32, o);
    } else {
#pragma unroll
      for (int i = 0; i < LB; ++i)
#pragma unroll
        for (int q = 0; q < 8; ++q) o[i][q] = 0;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i)
#pragma unroll
      for (int q = 0; q < 8; ++q) tile[i][kl * kPitch + 8 * g + q] = o[i][q];
  }
  __syncthreads();
  const int kq = threadIdx.x & 3, quad = (threadIdx.x >> 2) % (TN / 4);
  const int i = (threadIdx.x >> 2) / (TN / 4);  // limb
  const int64_t n = nb + 4 * quad;
  if (i >= LB || n >= N) return;
  int sum[4] = {0, 0, 0, 0};
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int k0 = 64 * h + 16 * kq;
    uint32_t o[4][4];  // [n][four k]
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint32_t r[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) r[j] = tile[i][(k0 + 4 * q + j) * kPitch + quad];
      o[0][q] = limb::bytes4<0>(r);
      o[1][q] = limb::bytes4<1>(r);
      o[2][q] = limb::bytes4<2>(r);
      o[3][q] = limb::bytes4<3>(r);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t at = LB == 1 && tiles
                             ? limb::chunk_tile(n + v, kb + k0, tiles)
                             : stacked_row(n + v, i, N, L) * ldk + kb + k0;
      if (n + v < N)
        *reinterpret_cast<uint4 *>(out + at) = make_uint4(o[v][0], o[v][1], o[v][2], o[v][3]);
#pragma unroll
      for (int q = 0; q < 4; ++q) sum[v] = sum4(o[v][q], sum[v]);
    }
  }
  if (!cadd) return;
  const int64_t live = i == 0 ? (K - kb < kCtK ? K - kb : kCtK) : 0;
#pragma unroll
  for (int v = 0; v < 4; ++v)
    commit_col((uint64_t)(int64_t)sum[v] << (8 * i), kq, n + v, N, live, alpha, beta, cadd);
}

// The tile of k_digit_cols_wide: 128 k x 64 n, pitch in bytes.
constexpr int kCtN = 64, kCtPitch = kCtN + 4;

// Digit i of the block's tile to out, a byte at a time, with the sum of this
// lane's 32 digits.
__device__ __forceinline__ int store_digit_cols(const uint8_t *tile, int64_t n, int nl, int kq,
                                                int i, int64_t N, int64_t kb, int64_t ldk, Limbs L,
                                                int8_t *__restrict__ out) {
  uint32_t o[8];
  int t = 0;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int k0 = 32 * kq + 4 * q;
    o[q] = (uint32_t)tile[k0 * kCtPitch + nl] | ((uint32_t)tile[(k0 + 1) * kCtPitch + nl] << 8) |
           ((uint32_t)tile[(k0 + 2) * kCtPitch + nl] << 16) |
           ((uint32_t)tile[(k0 + 3) * kCtPitch + nl] << 24);
    t = sum4(o[q], t);
  }
  uint4 *d = reinterpret_cast<uint4 *>(out + stacked_row(n, i, N, L) * ldk + kb + 32 * kq);
  d[0] = make_uint4(o[0], o[1], o[2], o[3]);
  d[1] = make_uint4(o[4], o[5], o[6], o[7]);
  return t;
}

// As k_digit_cols for fields of 33..64 bits: a limb of the tile at a time, each
// byte from its own field, four lanes to an n and 32 k.
__global__ __launch_bounds__(256) void k_digit_cols_wide(const uint32_t *__restrict__ w, int bits,
                                                         int sgn, int64_t K, int64_t N,
                                                         int64_t ldk, Limbs L,
                                                         int8_t *__restrict__ out, uint64_t alpha,
                                                         uint64_t beta,
                                                         int64_t *__restrict__ cadd) {
  __shared__ __align__(16) uint8_t tile[kCtK * kCtPitch];
  const int64_t nb = (int64_t)blockIdx.x * kCtN, kb = (int64_t)blockIdx.y * kCtK;
  const int t = threadIdx.x;
  const int nl = t >> 2, kq = t & 3;
  const int64_t n = nb + nl;
  uint64_t sum = 0;
  for (int i = 0; i < L.n; ++i) {
    const uint8_t flip = (uint8_t)limb::digit_flip(bits, sgn, i, L.n);
    for (int q = t; q < kCtK * kCtN; q += 256) {
      const int kl = q / kCtN, c = q % kCtN;
      const int64_t k = kb + kl, nn = nb + c;
      uint8_t d = 0;
      if (k < K && nn < N)
        d = (uint8_t)((uint64_t)value_at(w, (uint64_t)(k * N + nn), bits, sgn) >> (8 * i)) ^ flip;
      tile[kl * kCtPitch + c] = d;
    }
    __syncthreads();
    if (n < N)
      sum += (uint64_t)(int64_t)store_digit_cols(tile, n, nl, kq, i, N, kb, ldk, L, out)
             << (8 * i);
    __syncthreads();
  }
  if (cadd) commit_col(sum, kq, n, N, K - kb < kCtK ? K - kb : kCtK, alpha, beta, cadd);
}

hipError_t launch_digit_rows(const uint32_t *w, int bits, int sgn, int64_t M, int64_t K,
                             int64_t ldk, Limbs L, int8_t *out, uint64_t beta, int64_t *radd,
                             int64_t *cadd, int64_t N, hipStream_t s) {
  const uint64_t cap = cap_words32((uint64_t)M * (uint64_t)K, bits);
  switch (bits) {
#define CCM_DIGIT_ROWS(b)                                                                    \
  case b:                                                                                    \
    k_digit_rows<b><<<(unsigned)M, 256, 0, s>>>(w, cap, sgn, M, K, ldk, L, out, beta, radd,  \
                                                cadd, N);                                    \
    break;
    CCM_WIDTH_CASES_32(CCM_DIGIT_ROWS)
#undef CCM_DIGIT_ROWS
    default:
      k_digit_rows_wide<<<(unsigned)M, 256, 0, s>>>(w, bits, sgn, M, K, ldk, L, out, beta, radd,
                                                    cadd, N);
  }
  return hipGetLastError();
}

hipError_t launch_digit_cols(const uint32_t *w, int bits, int sgn, int64_t K, int64_t N,
                             int64_t ldk, Limbs L, int8_t *out, uint64_t alpha, uint64_t beta,
                             int64_t *cadd, int tiles, hipStream_t s) {
  const uint64_t cap = cap_words32((uint64_t)K * (uint64_t)N, bits);
  auto grid = [&](int tn) {
    return dim3((unsigned)((N + tn - 1) / tn), (unsigned)(ldk / kCtK));
  };
  // Wide tiles where they still give every CU two blocks: in us 42 (64 n) against
  // 27 (256) for 8192 x 8192 at 4 bits, but 6.8 against 9.1 (128) for 2000 x
  // 1801 at 10 bits and 3.8 against 6.6 for 10001 x 33 at 6.
  const int tw = ct_cols(limb::limbs_of(bits), true);
  const bool wide = (N + tw - 1) / tw * (ldk / kCtK) >= 512;
  switch (bits) {
#define CCM_DIGIT_COLS(b)                                                                     \
  case b: {                                                                                   \
    constexpr int narrow_n = ct_cols((b + 7) / 8, false), wide_n = ct_cols((b + 7) / 8, true); \
    auto k = wide ? k_digit_cols<b, wide_n> : k_digit_cols<b, narrow_n>;                      \
    k<<<grid(wide ? wide_n : narrow_n), 256, 0, s>>>(w, cap, sgn, K, N, ldk, L, out, alpha,   \
                                                     beta, cadd, tiles);                      \
    break;                                                                                    \
  }
    CCM_WIDTH_CASES_32(CCM_DIGIT_COLS)
#undef CCM_DIGIT_COLS
    default:
      k_digit_cols_wide<<<grid(kCtN), 256, 0, s>>>(w, bits, sgn, K, N, ldk, L, out, alpha, beta, cadd);
  }
  return hipGetLastError();
}

// The limbs of each operand per pass: every pair in one pass when one wave's
// accumulators hold them (at most 3 x 3, 4 x 2 or 2 x 4), otherwise the chunk
// sizes with the fewest passes.
void limb_chunks(int la, int lb, Limbs *A, Limbs *B) {
  int best = 1 << 20;
  for (int ca = 1; ca <= 4 && ca <= la; ++ca)
    for (int cb = 1; cb <= 4 && cb <= lb; ++cb) {
      if (!((ca <= 3 && cb <= 3) || (ca == 4 && cb <= 2) || (cb == 4 && ca <= 2))) continue;
      const int passes = ((la + ca - 1) / ca) * ((lb + cb - 1) / cb);
      if (passes < best) {
        best = passes;
        *A = Limbs{la, ca};
        *B = Limbs{lb, cb};
      }
    }
}

uint64_t up256(uint64_t n) { return (n + 255u) / 256u * 256u; }

// Scratch of the matrix-core path past the dense C: the digits of A, the
// digits of B^T, then the column and row addends where a digit offset asks
// for them.
struct LimbLayout {
  Limbs A, B;
  int64_t ldk;
  uint64_t alpha, beta;
  uint64_t b_at, cadd_at, radd_at, total;
};

LimbLayout limb_layout(int abits, int asgn, int bbits, int bsgn, int64_t M, int64_t K,
                       int64_t N) {
  LimbLayout p;
  limb_chunks(limb::limbs_of(abits), limb::limbs_of(bbits), &p.A, &p.B);
  p.ldk = padded_k(K);
  p.alpha = limb::digit_offset(abits, asgn);
  p.beta = limb::digit_offset(bbits, bsgn);
  const uint64_t a = (uint64_t)limb_rows(M, p.A.n) * (uint64_t)p.A.n * (uint64_t)p.ldk;
  const uint64_t b = (uint64_t)limb_rows(N, p.B.n) * (uint64_t)p.B.n * (uint64_t)p.ldk;
  p.b_at = a;  // rows are multiples of 128 bytes
  p.cadd_at = up256(a + b);
  p.radd_at = p.cadd_at + (p.alpha ? up256(8u * (uint64_t)N) : 0u);
  p.total = p.radd_at + (p.beta ? up256(8u * (uint64_t)M) : 0u);
  return p;
}

// Up to 256 columns, A is cheaper read packed once per group of columns (64 of
// them for A of three or four digits, 128 below; the second reading comes from
// the caches in part) than decoded to digits once.  us a product at 10000 x
// 10000, N = 256 / 257 (this form / digits): 6 x 4 bits 115 / 157, 8 x 6 133 /
// 205, 12 x 6 157 / 260, 20 x 6 295 / 402, 28 x 6 422 / 550; N = 33 (before: the
// digits, and the int64 path): 17 x 6 88 / 285 / 2290.
constexpr int64_t kNarrowCols = 256;

bool narrow_b(int abits, int bbits, int bsgn, int64_t N) {
  return abits <= 31 && bbits <= 8 && limb::digit_offset(bbits, bsgn) == 0 && N <= kNarrowCols;
}

// The narrow-B product: digits of B^T, the partial sums of the parts of K.
struct SkinnyLayout {
  int nb;     // 32-column blocks (0: not for this product)
  int waves;  // of a block of 16 rows (gemm_narrow.hpp; 0: gemm_skinny.hpp)
  int splits;
  int64_t ldk, kper;
  uint64_t part_at, total;
};

// A block takes as many columns of C as fit 128 accumulator registers a wave (L
// digits of A by nb blocks of 16).  `room` bounds the
// scratch (0: unbounded).
SkinnyLayout skinny_layout(int abits, int asgn, int bbits, int bsgn, int64_t M, int64_t K,
                           int64_t N, uint64_t room) {
  SkinnyLayout p = {};
  const int la = limb::limbs_of(abits);
  if (!narrow_b(abits, bbits, bsgn, N)) return p;
  p.nb = N <= 32 ? 1 : N <= 64 || la > 2 ? 2 : 4;
  const int64_t groups = (N + 32 * p.nb - 1) / (32 * p.nb);
  p.ldk = padded_k(K);
  const int64_t nk = p.ldk / limb::kBK;
  int64_t rows = (M + limb::kSkRows - 1) / limb::kSkRows * groups;
  int64_t slots = 4 * limb::sk_stage(abits, p.nb) <= 158 * 1024 ? 512 : 256;
  p.part_at = up256((uint64_t)N * (uint64_t)p.ldk);
  // Up to 64 columns in blocks of 16 rows (gemm_narrow.hpp), if the digits of whole
  // blocks of 16 columns fit the room.  us a plan, blocks of 128 rows / of 16, 17 x 6
  // bits: 1000 x 1000 x 33 32 / 25, 3000 x 3000 x 33 37 / 28, 500 x 20000 x 33 49 /
  // 32, 16000 x 4000 x 64 64 / 55, 10000 x 10001 x 33 83 / 81 (and without the sum of
  // the parts); past 48 columns the digits of B weigh as much as a large A, read
  // once per 16 rows: 10000 x 10001 x 64 86 / 89, 8192 x 8192 x 64 64 / 56.
  const uint64_t tiled = up256((uint64_t)((N + 15) / 16 * 16) * (uint64_t)p.ldk);
  const uint64_t abytes = (uint64_t)M * (uint64_t)K / 8 * (uint64_t)abits;
  if ((N <= 48 || (N <= 64 && abytes <= 160u << 20)) && (!room || tiled <= room)) {
    p.part_at = tiled;
    rows = (M + 15) / 16;
    p.waves = rows >= 512 ? 4 : 8;
    slots = 2048 / p.waves;
    const int64_t most = rows * (nk / p.waves);  // a step for every wave of a part
    slots = slots < most ? slots : most;
  }
  // parts of K until the blocks fill the chip once (two blocks per CU where
  // the LDS holds them)
  int64_t splits = rows < slots ? slots / rows : 1;
  splits = splits < nk ? splits : nk;
  const uint64_t one = 8u * (uint64_t)M * (uint64_t)N;
  if (room) {
    const uint64_t fit = room > p.part_at ? (room - p.part_at) / one : 0;
    if ((uint64_t)splits > fit) splits = fit < 2 ? 1 : (int64_t)fit;
  }
  p.kper = (nk + splits - 1) / splits;
  p.splits = (int)((nk + p.kper - 1) / p.kper);
  p.total = p.part_at + (p.splits > 1 ? up256((uint64_t)p.splits * one) : 0u);
  return p;
}

// Whether the launches of the two ways fit HIP's limits.
bool narrow_launches(const SkinnyLayout &p, int64_t M, int64_t N) {
  const uint64_t rows = p.waves ? 16 : limb::kSkRows, threads = p.waves ? 64 * p.waves : 512;
  return launch_fits(((uint64_t)M + rows - 1) / rows, threads) &&
         launch_fits(((uint64_t)N + 63) / 64, 256);
}

// Blocks of a pass over la x lb digits.
uint64_t limb_tiles(int la, int lb, int64_t M, int64_t N) {
  const int64_t tm = limb::tile_rows(la), tn = limb::tile_cols(la, lb);
  return (uint64_t)((M + tm - 1) / tm) * (uint64_t)((N + tn - 1) / tn);
}

bool limbs_launch(const LimbLayout &p, int64_t M, int64_t N) {
  bool ok = launch_fits((uint64_t)M, 256) && launch_fits(((uint64_t)N + 63) / 64, 256);
  for (int la : {p.A.n < p.A.chunk ? p.A.n : p.A.chunk, p.A.n % p.A.chunk})
    for (int lb : {p.B.n < p.B.chunk ? p.B.n : p.B.chunk, p.B.n % p.B.chunk})
      ok = ok && (!la || !lb || launch_fits(limb_tiles(la, lb, M, N), 512));
  return ok;
}

// C = the sum over the parts, and C's range.
template <typename OT>
__global__ __launch_bounds__(256) void k_sum_parts(const int64_t *__restrict__ part, int splits,
                                                   uint64_t mn, OT *__restrict__ C,
                                                   RangeSink sink) {
  int64_t lo = INT64_MAX, hi = INT64_MIN;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < mn; e += stride) {
    uint64_t v = 0;
    for (int q = 0; q < splits; ++q) v += (uint64_t)part[q * mn + e];
    const int64_t x = (int64_t)(OT)v;
    C[e] = (OT)x;
    lo = x < lo ? x : lo;
    hi = x > hi ? x : hi;
  }
  block_range_commit(lo, hi, 0, sink);
}

hipError_t launch_narrow(const SkinnyLayout &p, const uint32_t *aw, int abits, int asgn,
                         const uint32_t *bw, int bbits, int bsgn, int64_t M, int64_t K, int64_t N,
                         int out32, void *C, char *extra, RangeSink sink, hipStream_t s) {
  limb::SkinnyArgs a;
  hipError_t e = launch_digit_cols(bw, bbits, bsgn, K, N, p.ldk, Limbs{1, 1}, (int8_t *)extra, 0,
                                   0, nullptr, p.waves ? (int)((N + 15) / 16) : 0, s);
  if (e != hipSuccess) return e;
  a.aw = aw;
  a.cap_bytes = 4u * cap_words32((uint64_t)M * (uint64_t)K, abits);
  a.sgn = asgn;
  a.M = M;
  a.K = K;
  a.N = N;
  a.ldk = p.ldk;
  a.Bt = (const int8_t *)extra;
  a.kper = p.kper;
  a.splits = p.splits;
  a.part = (int64_t *)(extra + p.part_at);
  a.alpha = p.waves ? mt::tile_alpha(abits, asgn) : limb::digit_offset(abits, asgn);
  a.C = C;
  a.out32 = out32;
  a.sink = sink;
  if (p.waves) {
    switch (limb::limbs_of(abits)) {
      case 1: e = limb::launch_narrow_1(a, abits, p.waves, s); break;
      case 2: e = limb::launch_narrow_2(a, abits, p.waves, s); break;
      case 3: e = limb::launch_narrow_3(a, abits, p.waves, s); break;
      default: e = limb::launch_narrow_4(a, abits, p.waves, s);
    }
  } else {
    switch (limb::limbs_of(abits)) {
      case 1: e = limb::launch_skinny_1(a, abits, p.nb, s); break;
      case 2: e = limb::launch_skinny_2(a, abits, p.nb, s); break;
      case 3: e = limb::launch_skinny_3(a, abits, p.nb, s); break;
      default: e = limb::launch_skinny_4(a, abits, p.nb, s);
    }
  }
  if (e != hipSuccess || p.splits == 1) return e;
  const uint64_t mn = (uint64_t)M * (uint64_t)N;
  const uint64_t blocks = (mn + 255) / 256;
  const unsigned grid = (unsigned)(blocks < 2048 ? blocks : 2048);
  if (out32)
    k_sum_parts<int32_t><<<grid, 256, 0, s>>>(a.part, p.splits, mn, (int32_t *)C, sink);
  else
    k_sum_parts<int64_t><<<grid, 256, 0, s>>>(a.part, p.splits, mn, (int64_t *)C, sink);
  return hipGetLastError();
}

hipError_t launch_limbs(const uint32_t *aw, int abits, int asgn, const uint32_t *bw, int bbits,
                        int bsgn, int64_t M, int64_t K, int64_t N, int out32, void *C,
                        char *extra, RangeSink sink, hipStream_t s) {
  const LimbLayout p = limb_layout(abits, asgn, bbits, bsgn, M, K, N);
  int8_t *a8 = (int8_t *)extra, *b8 = (int8_t *)extra + p.b_at;
  int64_t *cadd = p.alpha ? (int64_t *)(extra + p.cadd_at) : nullptr;
  int64_t *radd = p.beta ? (int64_t *)(extra + p.radd_at) : nullptr;
  hipError_t e = launch_digit_rows(aw, abits, asgn, M, K, p.ldk, p.A, a8, p.beta, radd, cadd, N,
                                   s);
  if (e != hipSuccess) return e;
  e = launch_digit_cols(bw, bbits, bsgn, K, N, p.ldk, p.B, b8, p.alpha, p.beta, cadd, 0, s);
  if (e != hipSuccess) return e;
  const int64_t ar = limb_rows(M, p.A.n), br = limb_rows(N, p.B.n);
  for (int i0 = 0; i0 < p.A.n; i0 += p.A.chunk)
    for (int j0 = 0; j0 < p.B.n; j0 += p.B.chunk) {
      const int la = p.A.n - i0 < p.A.chunk ? p.A.n - i0 : p.A.chunk;
      const int lb = p.B.n - j0 < p.B.chunk ? p.B.n - j0 : p.B.chunk;
      const bool first = i0 == 0 && j0 == 0;
      const bool last = i0 + la == p.A.n && j0 + lb == p.B.n;
      // the overflow rule keeps the widths' sum low enough for this
      if (8 * (i0 + j0) >= 64) return hipErrorInvalidValue;
      limb::GemmArgs g;
      g.A = a8 + (int64_t)i0 * ar * p.ldk;
      g.Bt = b8 + (int64_t)j0 * br * p.ldk;
      g.arows = ar * la;
      g.brows = br * lb;
      g.M = M;
      g.N = N;
      g.ldk = p.ldk;
      g.C = C;
      g.radd = first ? radd : nullptr;
      g.cadd = first ? cadd : nullptr;
      g.shift = 8 * (i0 + j0);
      g.accumulate = first ? 0 : 1;
      g.sink = last ? sink : RangeSink{};
      e = limb::launch_pass(g, la, lb, out32, s);
      if (e != hipSuccess) return e;
    }
  return hipSuccess;
}

}  // namespace

namespace limb {

hipError_t launch_pass(const GemmArgs &p, int la, int lb, int out32, hipStream_t s) {
  switch (la) {
    case 1: return launch_pass_a1(p, lb, out32, s);
    case 2: return launch_pass_a2(p, lb, out32, s);
    case 3: return launch_pass_a3(p, lb, out32, s);
    case 4: return launch_pass_a4(p, lb, out32, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace limb

// Operands whose values fit int8 take no more scratch for a narrow B than for
// a wide one.
static SkinnyLayout narrow_layout(int abits, int asgn, int bbits, int bsgn, int64_t M, int64_t K,
                                  int64_t N, int i8) {
  const uint64_t room = i8 ? limb_layout(abits, asgn, bbits, bsgn, M, K, N).total : 0;
  return skinny_layout(abits, asgn, bbits, bsgn, M, K, N, room);
}

// Operands that fit in 32 bits are staged as int32 by the int64 path (products
// stay exact in int64); wider ones as int64.
static bool staged32(int abits, int asgn, int bbits, int bsgn) {
  return (abits < 32 || (abits == 32 && asgn)) && (bbits < 32 || (bbits == 32 && bsgn));
}

// Which way is the faster one: estimates of a plan's time in us, fitted to 3962
// products of M up to 2^20, N up to 4096 and K up to 10000 at nine pairs of widths,
// each timed both ways.  The int64 path walks K in chunks of 32, a block per 64 x
// 64 outputs; digits cost their launches, a block per row of A, tiles that a thin
// product leaves empty, and K padded to 128, so they lose where K is short (more
// so the taller A is) and win past it: 12 x 12 bits, int64 path / digits, 10000 x
// K x 10 at K = 97, 200, 1000 38 / 46, 53 / 49, 180 / 59; 10^5 x K x 10 at K = 200,
// 1000 116 / 194, 452 / 261; 2^20 x 16 x 16 159 / 1606; 10000 x K x 4096 at K = 32,
// 64, 128 115 / 165, 181 / 166, 322 / 169.  What the estimates choose takes at most
// 1.1 times as long as the int64 path, and 1.05 times as long as the faster way but
// for 58 of the products (up to 1.5 times).
static double int64_us(bool staged, int64_t M, int64_t K, int64_t N, double c_us) {
  const double tiles = (double)((M + kTM - 1) / kTM) * (double)((N + kTN - 1) / kTN);
  const double past = tiles > 128 ? tiles - 128 : 0;
  return 16 + (double)((K + kTK - 1) / kTK) * (staged ? 4.85 + 0.0068 * past : 7.6 + 0.0185 * past) +
         0.6 * c_us;
}

static double narrow_us(const SkinnyLayout &p, int la, int64_t M, int64_t N) {
  const double m = (double)M, steps = (double)(p.ldk / limb::kBK);
  if (p.waves) {
    const double nb = (double)((N + 15) / 16);
    return 21.2 + 0.06 * steps +
           m * (3.9e-5 + 7.9e-5 * nb + steps * la * (1.1e-5 + 1.57e-6 * nb));
  }
  const double nb = (double)((N + 31) / 32);
  return 27.9 + 0.23 * steps +
         m * (7.9e-5 + 3.6e-6 * (double)N + steps * la * (5.6e-6 + 6.7e-6 * nb));
}

static double limbs_us(const LimbLayout &p, int64_t M, int64_t N, double c_us) {
  const double steps = (double)(p.ldk / limb::kBK);
  double us = 21 + (double)M * (0.62 + 0.38 * p.A.n) * 1e-3 - c_us;
  for (int i = 0; i < p.A.n; i += p.A.chunk)
    for (int j = 0; j < p.B.n; j += p.B.chunk) {
      const int la = p.A.n - i < p.A.chunk ? p.A.n - i : p.A.chunk;
      const int lb = p.B.n - j < p.B.chunk ? p.B.n - j : p.B.chunk;
      // a wave stores its part of the block's tile, less what lies past C
      const bool tall = lb >= 3 && la < 3;
      const double wm = limb::tile_rows(la) / (tall ? 4 : 2);
      const double wn = limb::tile_cols(la, lb) / (tall ? 2 : 4);
      const double store = 21. / 8192 * (M < wm ? M : wm) * wn * (0.4 + (N < wn ? 0.6 * N / wn : 0.6));
      const double turns = (double)limb_tiles(la, lb, M, N) / 256;
      us += (turns > 1 ? turns : 1) * (5.7 + store + 1.7 * steps) + 1.9 * c_us;  // C read and written
    }
  return us;
}

uint64_t matmul_fast_bytes(int abits, int asgn, int bbits, int bsgn, int64_t M, int64_t K,
                           int64_t N, int i8, int out32) {
  const int64_t ldk = padded_k(K);
  // Six digits and a C that fits int32: outer products of signed operands (a field
  // of b bits may hold no magnitude past 2^(b-2), so 17 by 17 bits can stay below
  // 2^31) and products by a matrix of zeros.
  if (out32 && limb::limbs_of(abits) + limb::limbs_of(bbits) >= 6) return 0;
  if ((ldk >= (1 << 17) && !i8) || ldk / kCtK > 65535) return 0;  // int32 sums, grid rows
  const LimbLayout p = limb_layout(abits, asgn, bbits, bsgn, M, K, N);
  const SkinnyLayout n = narrow_layout(abits, asgn, bbits, bsgn, M, K, N, i8);
  const bool narrow = n.nb && narrow_launches(n, M, N);
  if (i8) {
    // one launch against three, for one wave of the int64 path's blocks
    if (!n.nb && K <= 96 && M <= (1 << 20) && N <= (1 << 20) && M * N <= (1 << 20)) return 0;
    return narrow || limbs_launch(p, M, N) ? p.total : 0;
  }
  const double c_us = (out32 ? 4. : 8.) * (double)M * (double)N / 5e6;  // C at 5 TB/s
  const double other = int64_us(staged32(abits, asgn, bbits, bsgn), M, K, N, c_us);
  if (n.nb) return narrow && narrow_us(n, p.A.n, M, N) <= other ? n.total : 0;
  return limbs_launch(p, M, N) && limbs_us(p, M, N, c_us) <= other ? p.total : 0;
}

hipError_t launch_matmul(const uint32_t *aw, int abits, int asgn, const uint32_t *bw,
                         int bbits, int bsgn, int64_t M, int64_t K, int64_t N, int i8, int out32,
                         void *scratch, uint64_t c_bytes, uint64_t scratch_bytes, RangeSink sink,
                         hipStream_t s) {
  const uint64_t fast = matmul_fast_bytes(abits, asgn, bbits, bsgn, M, K, N, i8, out32);
  if (fast && scratch_bytes >= c_bytes && scratch_bytes - c_bytes >= fast) {
    const SkinnyLayout n = narrow_layout(abits, asgn, bbits, bsgn, M, K, N, i8);
    const bool aligned = (uintptr_t)aw % 16 == 0;  // 16-byte copies of the payload itself
    if (n.nb && aligned && narrow_launches(n, M, N))
      return launch_narrow(n, aw, abits, asgn, bw, bbits, bsgn, M, K, N, out32, scratch,
                           (char *)scratch + c_bytes, sink, s);
    // the scratch of a narrow product past int8 is that form's alone
    if ((!n.nb || i8) && limbs_launch(limb_layout(abits, asgn, bbits, bsgn, M, K, N), M, N))
      return launch_limbs(aw, abits, asgn, bw, bbits, bsgn, M, K, N, out32, scratch,
                          (char *)scratch + c_bytes, sink, s);
  }
  if (staged32(abits, asgn, bbits, bsgn))
    return launch_generic<int32_t>(aw, abits, asgn, bw, bbits, bsgn, M, K, N, out32, scratch,
                                   sink, s);
  return launch_generic<int64_t>(aw, abits, asgn, bw, bbits, bsgn, M, K, N, out32, scratch,
                                 sink, s);
}

}  // namespace ccm
