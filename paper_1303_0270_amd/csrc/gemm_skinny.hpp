// C = A B for a B of 65 to 256 columns, or 49 and more by a large A (narrower ones:
// gemm_narrow.hpp; also those whose scratch has no room for it): A is read once, packed,
// and its digits are made in registers on the way into the matrix cores.
//
// With few columns of C the product is bound by reading A, not by the
// products, so decoding A to digits in memory first (packed bytes in, L bytes
// an element out and in again) and multiplying 256-column tiles costs several
// times the read.  Here a block owns 128 rows (32 per pair of waves, the rows
// of an MFMA operand) and up to 128 columns over one part of K.
//   * Per step of 128 columns of A, the 16-byte chunks that cover the pair's 32
//     row segments are copied into LDS (memory-to-LDS copies, consecutive
//     lanes on consecutive chunks of a row) while the previous step is
//     multiplied; a step advances every row by exactly 16 B bytes, so a lane's
//     offsets are fixed.  An odd number of chunks per row keeps the lanes'
//     word reads (one row each) at most two to a bank.
//   * A sum over K may take its terms in any order, so lane half h takes the
//     64 columns 64 h.. of the step, as two groups of 32 whose fields sit at
//     compile-time offsets after one funnel shift per word (rows start at any
//     bit): 16 columns of each half make one 32-deep MFMA.  The two waves of a
//     pair take one group each: a step's LDS holds one block per CU for wide
//     A, and a single wave per SIMD left every LDS read and MFMA exposed.
//     Their sums are added through LDS at the end.
//   * The digits of B, zero past K, are staged beside A in the same order; the
//     column sums that A's digit offset needs are taken from them on the way.
// Measured at 17 x 6 bits, 10000 x 10001 x 33 (213 MB of A): 61-64 us, 3.4
// TB/s, against 252 us for A's digits written and multiplied (126 + 126) and
// 2250 us for the int64 path; one wave per 32 rows took 72 us.
//   * K is split over blocks until they fill the chip once; the parts' 64-bit
//     sums are added by a second kernel, which also folds the range.  A single
//     part stores C itself.
#pragma once

#include "gemm_limb.hpp"

namespace ccm {
namespace limb {

constexpr int kSkThreads = 512;

template <int B, int NB>
__global__ __launch_bounds__(kSkThreads) void k_gemm_skinny(SkinnyArgs p) {
  constexpr int L = (B + 7) / 8, CH = sk_chunks(B), AI = sk_insts(B);
  constexpr int kStage = sk_stage(B, NB);
  extern __shared__ __align__(16) int8_t sk_lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pair = wave & 3, grp = wave >> 2;  // 32 rows; which group of each half
  const int64_t m0 = (int64_t)blockIdx.x * kSkRows + 32 * pair;
  const int64_t n0 = (int64_t)blockIdx.z * (32 * NB);
  const int64_t c0 = (int64_t)blockIdx.y * p.kper;  // first K step of this part
  const int64_t nsteps = p.ldk / kBK;
  const int64_t c1 = c0 + p.kper < nsteps ? c0 + p.kper : nsteps;

  // bit of (row, first column of the part); rows past M repeat the last one
  // (their results are not stored)
  auto row_bit = [&](int r) {
    int64_t row = m0 + r;
    row = row < p.M ? row : p.M - 1;
    return ((uint64_t)row * (uint64_t)p.K + (uint64_t)c0 * kBK) * B;
  };
  const uint64_t base = row_bit(0) / 128 * 16;  // bytes; the pair's rows follow within 2^31
  // the pair's copies alternate between its waves
  constexpr int AH = (AI + 1) / 2;
  uint32_t aoff[AH];
#pragma unroll
  for (int i = 0; i < AH; ++i) {
    int q = (2 * i + grp) * 64 + lane;
    q = q < 32 * CH ? q : 32 * CH - 1;
    aoff[i] = (uint32_t)(row_bit(q / CH) / 128 * 16 - base) + 16 * (q % CH);
  }
  const int brow = lane / 8, bpos = lane % 8;
  auto stage = [&](int64_t c, int buf) {
    int8_t *dst = sk_lds + buf * kStage;
    const uint64_t at = base + (uint64_t)(c - c0) * (16 * B);
    // chunks wholly past the payload hold no field of A: read its end instead
    const uint64_t end = p.cap_bytes - 16;
    const uint64_t from = at < end ? at : end;
    const uint32_t lim = end - from < 0xfffffff0u ? (uint32_t)(end - from) : 0xfffffff0u;
    const int8_t *src = (const int8_t *)p.aw + from;
#pragma unroll
    for (int i = 0; i < AH; ++i) {
      if (2 * i + grp < AI) {
        const uint32_t o = aoff[i] < lim ? aoff[i] : lim;
        __builtin_amdgcn_global_load_lds(
            (const void *)(src + o),
            (__attribute__((address_space(3))) void *)(dst + (pair * AI + 2 * i + grp) * 1024), 16,
            0, 0);
      }
    }
    dst += 4 * AI * 1024;
#pragma unroll
    for (int q = 0; q < (NB + 1) / 2; ++q) {
      const int I = wave + 8 * q;  // 8 rows of the 32 NB
      if (I < 4 * NB) {
        const int r = I * 8 + brow;
        const int64_t gr = n0 + r < p.N ? n0 + r : p.N - 1;
        __builtin_amdgcn_global_load_lds(
            (const void *)(p.Bt + gr * p.ldk + c * kBK + 16 * (bpos ^ swz(r))),
            (__attribute__((address_space(3))) void *)(dst + I * 1024), 16, 0, 0);
      }
    }
  };

  v16i acc[L][NB];
  int csum[NB];
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    csum[t] = 0;
#pragma unroll
    for (int i = 0; i < L; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][t][r] = 0;
  }

  const int half = lane >> 5;
  const uint64_t bit = row_bit(lane & 31);
  const int sh = (int)(bit & 31);
  const int word = (lane & 31) * CH * 4 + (int)((bit & 127) >> 5) + half * 2 * B + grp * B;

  if (c0 < c1) stage(c0, 0);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  for (int64_t c = c0; c < c1; ++c) {
    const int cur = (int)((c - c0) & 1);
    if (c + 1 < c1) stage(c + 1, cur ^ 1);  // in flight during this step
    const uint32_t *aw = reinterpret_cast<const uint32_t *>(sk_lds + cur * kStage + pair * AI * 1024);
    const int8_t *bt = sk_lds + cur * kStage + 4 * AI * 1024;
    uint32_t ww[B + 1];
#pragma unroll
    for (int q = 0; q <= B; ++q) ww[q] = aw[word + q];
    v4i b[2][NB];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int t = 0; t < NB; ++t) {
        const int r = t * 32 + (lane & 31);
        b[j][t] = *reinterpret_cast<const v4i *>(bt + r * kBK +
                                                 16 * ((4 * half + 2 * grp + j) ^ swz(r)));
      }
#pragma unroll
    for (int q = 0; q < B; ++q) ww[q] = __builtin_amdgcn_alignbit(ww[q + 1], ww[q], sh);
    uint32_t o[L][8];
    words_digits<B>(ww, p.sgn, o);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if constexpr (L > 1 || B == 8) {
#pragma unroll
        for (int t = 0; t < NB; ++t)
#pragma unroll
          for (int q = 0; q < 4; ++q) csum[t] = sum4((uint32_t)b[j][t][q], csum[t]);
      }
#pragma unroll
      for (int i = 0; i < L; ++i) {
        const v4i a = {(int)o[i][4 * j], (int)o[i][4 * j + 1], (int)o[i][4 * j + 2],
                       (int)o[i][4 * j + 3]};
#pragma unroll
        for (int t = 0; t < NB; ++t)
          acc[i][t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b[j][t], acc[i][t], 0, 0, 0);
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();  // the next step has landed and this buffer is read
  }

  // digits combined, the offset's column sums added, then the pair's two waves
  int64_t lo = INT64_MAX, hi = INT64_MIN;
  int64_t *part = p.part + (int64_t)blockIdx.y * p.M * p.N;
  int64_t *xch = reinterpret_cast<int64_t *>(sk_lds) + pair * 16 * 64 + lane;
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    const int64_t n = n0 + t * 32 + (lane & 31);
    const uint64_t add =
        p.alpha * (uint64_t)(int64_t)(csum[t] + __shfl_xor(csum[t], 32, 64));
    uint64_t v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      v[r] = add;
#pragma unroll
      for (int i = 0; i < L; ++i) v[r] += (uint64_t)(int64_t)acc[i][t][r] << (8 * i);
    }
    if (grp == 1) {
#pragma unroll
      for (int r = 0; r < 16; ++r) xch[64 * r] = (int64_t)v[r];
    }
    __syncthreads();
    if (grp == 0) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t m = m0 + 8 * (r / 4) + 4 * half + r % 4;
        v[r] += (uint64_t)xch[64 * r];
        if (m < p.M && n < p.N) {
          const int64_t at = m * p.N + n;
          if (p.splits > 1) {
            part[at] = (int64_t)v[r];
          } else {
            const int64_t x = p.out32 ? (int64_t)(int32_t)v[r] : (int64_t)v[r];
            if (p.out32)
              ((int32_t *)p.C)[at] = (int32_t)x;
            else
              ((int64_t *)p.C)[at] = x;
            lo = x < lo ? x : lo;
            hi = x > hi ? x : hi;
          }
        }
      }
    }
    __syncthreads();  // the exchange is read before the next block's values
  }
  if (p.splits == 1) block_range_commit(lo, hi, 0, p.sink);
}

template <int B, int NB>
hipError_t launch_skinny_one(const SkinnyArgs &p, hipStream_t s) {
  // two steps, and the exchange of the pairs' sums
  constexpr int lds = 2 * sk_stage(B, NB) > 32768 ? 2 * sk_stage(B, NB) : 32768;
  static_assert(lds <= 160 * 1024 - 1024, "LDS");
  auto kern = k_gemm_skinny<B, NB>;
  static const hipError_t attr = hipFuncSetAttribute(
      reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  (void)attr;
  const dim3 grid((unsigned)((p.M + kSkRows - 1) / kSkRows), (unsigned)p.splits,
                  (unsigned)((p.N + 32 * NB - 1) / (32 * NB)));
  kern<<<grid, kSkThreads, lds, s>>>(p);
  return hipGetLastError();
}

template <int B>
hipError_t launch_skinny_b(const SkinnyArgs &p, int nb, hipStream_t s) {
  if constexpr (B <= 8) {  // up to 32 columns: int8 pairs with no room for chunk tiles
    if (nb == 1) return launch_skinny_one<B, 1>(p, s);
  }
  if (nb == 2) return launch_skinny_one<B, 2>(p, s);
  if constexpr (B <= 16) {
    if (nb == 4) return launch_skinny_one<B, 4>(p, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace limb
}  // namespace ccm
