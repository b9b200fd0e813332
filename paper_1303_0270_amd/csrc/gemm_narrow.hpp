// C = A B for at most 64 columns of B of one digit: a tile of 16 rows of A per
// block, every wave on its own steps of K, no barrier until their sums meet.
//
// As in gemm_skinny.hpp, A is read once, packed, and its digits are made in
// registers; what differs is that nothing is shared while K is walked:
//   * Wave v of W takes the steps (128 columns of A) v, v + W, ... of the block's
//     part of K: the waves read 16 W B consecutive bytes of each row, and no step
//     waits for another wave's copies.
//   * A step's row segments (the 16-byte chunks that cover them, an odd count so
//     that the rows' word reads lie apart) are copied into the wave's one LDS
//     buffer; its words go to registers at once, and the next step's copies are
//     in flight while they are decoded (as in mv_tile.hpp).
//   * The digits of B come straight from memory into the operand registers, in
//     flight while A's are made: 48 columns are 6 KB a step, which the L2s hold.
//     They are stored in chunk tiles, in the order of the lanes: from rows of
//     digits, four lanes of a load took four lines, and the loads set the time
//     (64 columns at 8 bits, 10000 x 10001: a plan took 82 us, 54 now).
//   * v_mfma_i32_16x16x64_i8: 16 rows by blocks of 16 columns, so 33 columns cost
//     48, and three digits by 64 columns take 48 accumulator registers.  Lane
//     (r, h) = (lane % 16, lane / 16) holds group h (32 columns) of row r's step,
//     which feeds two MFMAs of 16 bytes; the columns of B lie the same way.
// Bound by reading A and, from 33 columns, by the digits of B (a wave reads them
// for 16 rows).  17 x 6 bits, 10000 x 10001 x 33 (213 MB of A): 66 us, 3.2 TB/s, and
// one part of K, where gemm_skinny.hpp took 62 and the sum of its parts 8.5; 45 at
// 16 columns.  A plan of 1000 x 1000 x 33 24.5 us (32.4), 8192 x 8192 x 33 52.6 (61).
// Two buffers a wave, and the digits of B a step ahead, measured no faster.
#pragma once

#include "gemm_limb.hpp"
#include "mv_tile.hpp"

namespace ccm {
namespace limb {

constexpr int kNwWaves = 8;  // at most
constexpr int nw_chunks(int B) { return (B + 2) | 1; }
constexpr int nw_insts(int B) { return (16 * nw_chunks(B) + 63) / 64; }

template <int B, int NB>
__global__ __launch_bounds__(64 * kNwWaves) void k_gemm_narrow(SkinnyArgs p) {
  constexpr int L = (B + 7) / 8, CH = nw_chunks(B), AI = nw_insts(B);
  extern __shared__ __align__(16) int8_t nw_lds[];
  typedef const __attribute__((address_space(1))) int8_t *global_bytes;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int waves = blockDim.x >> 6;
  const int n = lane & 15, h = lane >> 4;
  const int64_t m0 = (int64_t)blockIdx.x * 16;
  const int64_t nsteps = p.ldk / kBK;
  const int64_t c0 = (int64_t)blockIdx.y * p.kper;  // first K step of this part
  const int64_t c1 = c0 + p.kper < nsteps ? c0 + p.kper : nsteps;

  // bit of (row, first column of the part); rows past M repeat the last one
  // (their results are not stored)
  auto row_bit = [&](int r) {
    int64_t row = m0 + r;
    row = row < p.M ? row : p.M - 1;
    return ((uint64_t)row * (uint64_t)p.K + (uint64_t)c0 * kBK) * B;
  };
  const uint64_t base = row_bit(0) / 128 * 16;
  uint32_t aoff[AI];
#pragma unroll
  for (int i = 0; i < AI; ++i) {
    int q = i * 64 + lane;
    q = q < 16 * CH ? q : 16 * CH - 1;
    aoff[i] = (uint32_t)(row_bit(q / CH) / 128 * 16 - base) + 16 * (q % CH);
  }
  int8_t *buf = nw_lds + wave * AI * 1024;
  const global_bytes aw = (global_bytes)(uintptr_t)p.aw;
  auto stage = [&](int64_t c) {
    // this wave's reads of the buffer have returned
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    const uint64_t at = base + (uint64_t)(c - c0) * (16 * B), end = p.cap_bytes - 16;
    // chunks wholly past the payload hold no field of A: read its end instead
    const uint64_t from = at < end ? at : end;
    const uint32_t lim = end - from < 0xfffffff0u ? (uint32_t)(end - from) : 0xfffffff0u;
#pragma unroll
    for (int i = 0; i < AI; ++i) {
      const uint32_t o = aoff[i] < lim ? aoff[i] : lim;
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void *)(aw + from + o),
          (__attribute__((address_space(3))) void *)(buf + i * 1024), 16, 0, 0);
    }
  };
  const int8_t *bt = p.Bt + 16 * lane;  // chunk tiles: 1 KB per step, block of 16 columns and MFMA
  v4i acc[L][NB];
  int csum[NB];
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    csum[t] = 0;
#pragma unroll
    for (int i = 0; i < L; ++i) acc[i][t] = v4i{0, 0, 0, 0};
  }
  const uint64_t bit = row_bit(n);
  const int sh = (int)(bit & 31u);
  const int word = n * CH * 4 + (int)((bit & 127u) >> 5) + h * B;

  const uint32_t flip = mt::top_flip(B, p.sgn);
  if (c0 + wave < c1) stage(c0 + wave);
  for (int64_t c = c0 + wave; c < c1; c += waves) {
    v4i b[2][NB];
#pragma unroll
    for (int t = 0; t < NB; ++t)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        b[j][t] = *reinterpret_cast<const v4i *>(bt + ((c * NB + t) * 2 + j) * 1024);
    // this step's copies, which are older than B's loads (all issued by here)
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(%0)" ::"i"(2 * NB) : "memory");
    const uint32_t *wp = reinterpret_cast<const uint32_t *>(buf);
    uint32_t ww[B + 1];
#pragma unroll
    for (int q = 0; q <= B; ++q) ww[q] = wp[word + q];
    // The next step's copies, while this one is decoded (past the last one, this
    // one again: a branch here would make B's wait one for the copies too).
    stage(c + waves < c1 ? c + waves : c);
#pragma unroll
    for (int q = 0; q < B; ++q) ww[q] = __builtin_amdgcn_alignbit(ww[q + 1], ww[q], sh);
    uint32_t o[L][8];
    mt::tile_digits<B, false>(ww, flip, o);
#pragma unroll
    for (int t = 0; t < NB; ++t)
#pragma unroll
      for (int q = 0; q < 8; ++q) csum[t] = sum4((uint32_t)b[q / 4][t][q % 4], csum[t]);
#pragma unroll
    for (int i = 0; i < L; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const v4i a = {(int)o[i][4 * j], (int)o[i][4 * j + 1], (int)o[i][4 * j + 2],
                       (int)o[i][4 * j + 3]};
#pragma unroll
        for (int t = 0; t < NB; ++t)
          acc[i][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b[j][t], acc[i][t], 0, 0, 0);
      }
  }

  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the copies past the last step

  // The digits combined, the offset's column sums added, the waves' sums through
  // LDS: lane (n, h) holds column 16 t + n of rows 4 h .. 4 h + 3.
  int64_t lo = INT64_MAX, hi = INT64_MIN;
  uint64_t *red = reinterpret_cast<uint64_t *>(nw_lds);
  int64_t *part = p.part + (int64_t)blockIdx.y * p.M * p.N;
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    int cs = csum[t];
    cs += __shfl_xor(cs, 16, 64);
    cs += __shfl_xor(cs, 32, 64);
    const uint64_t add = p.alpha * (uint64_t)(int64_t)cs;
    __syncthreads();  // the buffers, or the sums before, are read
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      uint64_t v = add;
#pragma unroll
      for (int i = 0; i < L; ++i) v += (uint64_t)(int64_t)acc[i][t][r] << (8 * i);
      red[(wave * 4 + r) * 64 + lane] = v;
    }
    __syncthreads();
    if (tid < 256) {
      uint64_t v = 0;
      for (int q = 0; q < waves; ++q) v += red[q * 256 + tid];
      const int64_t m = m0 + 4 * h + (tid >> 6), col = 16 * t + n;
      if (m < p.M && col < p.N) {
        const int64_t at = m * p.N + col;
        if (p.splits > 1) {
          part[at] = (int64_t)v;
        } else {
          const int64_t x = p.out32 ? (int64_t)(int32_t)v : (int64_t)v;
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
  if (p.splits == 1) block_range_commit(lo, hi, 0, p.sink);
}

template <int B>
hipError_t launch_narrow_b(const SkinnyArgs &p, int waves, hipStream_t s) {
  const dim3 grid((unsigned)((p.M + 15) / 16), (unsigned)p.splits);
  // the waves' buffers, then their sums of 16 x 16 of C
  const size_t lds = (size_t)waves * (nw_insts(B) > 2 ? nw_insts(B) : 2) * 1024;
  static_assert(kNwWaves * nw_insts(B) <= 160, "LDS");
  static const hipError_t attr = [] {
    hipError_t e = hipSuccess;
    for (auto k : {k_gemm_narrow<B, 1>, k_gemm_narrow<B, 2>, k_gemm_narrow<B, 3>,
                   k_gemm_narrow<B, 4>}) {
      const hipError_t f = hipFuncSetAttribute(
          reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024);
      e = e != hipSuccess ? e : f;
    }
    return e;
  }();
  (void)attr;
  auto k = p.N <= 16   ? k_gemm_narrow<B, 1>
           : p.N <= 32 ? k_gemm_narrow<B, 2>
           : p.N <= 48 ? k_gemm_narrow<B, 3>
                       : k_gemm_narrow<B, 4>;
  k<<<grid, 64 * waves, lds, s>>>(p);
  return hipGetLastError();
}

}  // namespace limb
}  // namespace ccm
