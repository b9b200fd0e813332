// Row tiles of y = A x on matrix cores: 16 rows of packed fields by the base-256
// digits of x.
//
// A matvec leaves the matrix cores nothing to reuse, but they take over what
// the vector units otherwise spend most of their instructions on: the
// products, the sums along a row and the sums across its lanes.  What is left
// per field is its way into a byte (extract and pack, or a shift and a mask for
// four fields at widths that divide a byte).
//
//   * A field's digits are those of the products on matrix cores
//     (gemm_limb.hpp), signed fields as unsigned ones with the top bit flipped:
//     a = alpha + sum_i d_i 256^i, d_i in [-128, 127], L = ceil(b / 8) digits.
//   * x (int32) is staged in LDS as D = 4 digit rows: lower digits byte - 128, the
//     top one the signed top byte, and a row of ones:
//     x_k = X0 + sum_n e_n(k) 256^n with X0 = 128 sum_{n < D-1} 256^n.  Past the
//     last column every row is zero, whatever the fields read there.
//   * v_mfma_i32_16x16x64_i8 multiplies 16 rows of A by these D + 1 columns (of
//     16: the others get weight 0).  Column n of row m holds sum_k d_i e_n, so
//     y_m = sum_n w_n sum_i 256^i S_in + alpha sum_k x_k mod 2^64 with
//     w_n = 256^n, w_D = X0.  int32 sums are exact up to 2^17 columns.
//   * A step is 128 columns: lane (r, h) = (lane % 16, lane / 16) owns group h of
//     row r, 32 fields at compile-time offsets after one funnel shift per word,
//     which feed two MFMAs (16 bytes each).  The order of a group's fields in
//     those bytes is the digit rows' order too, so at b = 1, 2 and 4 it is the
//     one that shifts and masks give.
#pragma once

#include "ccm_internal.hpp"
#include "gemm_limb.hpp"
#include "group_codec.hpp"

namespace ccm {
namespace mt {

using limb::v4i;

// Pointers that a kernel reads from memory are of no known address space, and
// loads through them (flat) count as LDS operations too: every wait for an LDS
// read would wait for the words in flight.  These say that they are global.
template <typename T>
using global_ptr = const __attribute__((address_space(1))) T *;
template <typename T>
__device__ __forceinline__ global_ptr<T> as_global(const T *p) {
  return (global_ptr<T>)(uintptr_t)p;
}

constexpr int kTileRows = 16;
constexpr int kStep = 128;  // columns per step: four groups

// Fields whose bytes a shift and a mask give are taken 8 / b apart.
__host__ __device__ constexpr int spread_of(int b) {
  return b == 1 || b == 2 || b == 4 ? 8 / b : 1;
}

// XOR of four top digits, and alpha, of fields of `bits` bits.
__device__ __forceinline__ uint32_t top_flip(int bits, int sgn) {
  const int t = bits - 8 * (limb::limbs_of(bits) - 1);  // bits in the top byte
  const uint32_t f = sgn ? (t == 8 ? 0u : 1u << (t - 1)) : (t == 8 ? 0x80u : 0u);
  return f * 0x01010101u;
}
__host__ __device__ inline uint64_t tile_alpha(int bits, int sgn) {
  const int L = limb::limbs_of(bits), t = bits - 8 * (L - 1);
  uint64_t a = 0;
  for (int i = 0; i + 1 < L; ++i) a += 128ull << (8 * i);
  if (!sgn && t == 8) a += 128ull << (8 * (L - 1));
  if (sgn && t < 8) a -= 1ull << (8 * (L - 1) + t - 1);
  return a;
}

// Digits of 32 fields of B <= 32 bits from their aligned words; SPREAD: in the
// order of spread_of(B), otherwise as they follow each other.
template <int B, bool SPREAD = true>
__device__ __forceinline__ void tile_digits(const uint32_t *ww, uint32_t flip,
                                            uint32_t (&o)[(B + 7) / 8][8]) {
  constexpr int L = (B + 7) / 8;
  if constexpr (SPREAD && spread_of(B) > 1) {
    constexpr int S = 8 / B;
    constexpr uint32_t mask = B == 1 ? 0x01010101u : B == 2 ? 0x03030303u : 0x0f0f0f0fu;
#pragma unroll
    for (int q = 0; q < 8; ++q) o[0][q] = (ww[q / S] >> (B * (q % S))) & mask;
  } else if constexpr (B == 8) {
#pragma unroll
    for (int q = 0; q < 8; ++q) o[0][q] = ww[q];
  } else if constexpr (B == 16) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      o[0][q] = __builtin_amdgcn_perm(ww[2 * q + 1], ww[2 * q], 0x06040200u);
      o[1][q] = __builtin_amdgcn_perm(ww[2 * q + 1], ww[2 * q], 0x07050301u);
    }
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      uint32_t v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = codec::field32<B, false>(ww, 4 * q + i);
      o[0][q] = limb::bytes4<0>(v);
      if constexpr (L > 1) o[1][q] = limb::bytes4<1>(v);
      if constexpr (L > 2) o[2][q] = limb::bytes4<2>(v);
      if constexpr (L > 3) o[3][q] = limb::bytes4<3>(v);
    }
  }
#pragma unroll
  for (int q = 0; q < 8; ++q) {
#pragma unroll
    for (int i = 0; i < L - 1; ++i) o[i][q] ^= 0x80808080u;
    o[L - 1][q] ^= flip;
  }
}

// Digit rows of x in LDS: row n at n * pitch, columns padded to whole steps; a
// pitch off the bank period keeps the rows' reads apart.
__host__ __device__ constexpr int x_pitch(int cols) {
  return (cols + kStep - 1) / kStep * kStep + 16;
}
constexpr int kXDigits = 4;
constexpr int x_lds(int cols) { return (kXDigits + 1) * x_pitch(cols); }
constexpr uint64_t x_offset() {
  uint64_t a = 0;
  for (int n = 0; n + 1 < kXDigits; ++n) a += 128ull << (8 * n);
  return a;
}

// Stages cols values of x in the field order of `spread`, NT threads; returns
// this thread's share of their sum (mod 2^64).  A thread makes one word (four
// columns) of every digit row at a time, `UNR` of them with their loads in
// flight together.
template <int NT>
__device__ __forceinline__ uint64_t stage_x(const int32_t *__restrict__ xp, int cols, int spread,
                                            uint8_t *lds) {
  constexpr int D = kXDigits, UNR = 2;
  const global_ptr<int32_t> x = as_global(xp);
  const int pitch = x_pitch(cols), nw = (pitch - 16) / 4;
  uint64_t sum = 0;
  for (int t0 = threadIdx.x; t0 < nw; t0 += NT * UNR) {
    int32_t v[UNR][4];
    uint32_t ones[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int t = t0 + u * NT, s = t & 7;
      const int e = (t & ~7) * 4 + s / spread * (4 * spread) + s % spread;
      ones[u] = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int c = e + spread * i;
        v[u][i] = x[c < cols ? c : cols - 1];
        if (c < cols) ones[u] |= 1u << (8 * i);
      }
    }
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int t = t0 + u * NT;
      if (t >= nw) break;
      const uint32_t live = ones[u] * 0xffu;
      uint32_t b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        b[i] = (uint32_t)v[u][i];
        if (ones[u] >> (8 * i) & 1u) sum += (uint64_t)(int64_t)v[u][i];
      }
      const uint32_t w[D] = {limb::bytes4<0>(b), limb::bytes4<1>(b), limb::bytes4<2>(b),
                             limb::bytes4<3>(b)};
#pragma unroll
      for (int n = 0; n < D; ++n)
        *reinterpret_cast<uint32_t *>(lds + n * pitch + 4 * t) =
            (w[n] ^ (n < D - 1 ? 0x80808080u : 0u)) & live;
      *reinterpret_cast<uint32_t *>(lds + D * pitch + 4 * t) = ones[u];
    }
  }
  return sum;
}

// A unit of a tile's work: `steps` steps of its 16 rows, copied into LDS as the
// 16-byte chunks that cover each row's segment (up to 15 bytes before it and
// the word after it; an odd count keeps the rows' word reads apart).  A unit's
// words are held in registers: steps as far as those of a wide field go.
template <int B>
struct Unit {
  static constexpr int steps = B <= 4 ? 4 : B <= 12 ? 2 : 1;
  static constexpr int chunks = (B * steps + 2) | 1;
  static constexpr int insts = (kTileRows * chunks + 63) / 64;  // copies per lane
  static constexpr int bytes = 1024 * insts;
};
constexpr int unit_bytes(int b) {
  switch (b) {
#define CCM_UNIT(n) \
  case n: return Unit<n>::bytes;
    CCM_WIDTH_CASES_32(CCM_UNIT)
#undef CCM_UNIT
    default: return 0;
  }
}

// y of the tiles of one wave of `waves` (tile t: rows row0 + 16 t.., below row_end;
// ntile of them, dealt in turn), over the staged columns of the matrix.
//   * Rows are read through LDS (buf: a unit of the wave's own): lanes that own a
//     group each would touch 64 lines with every load, and the waves of a CU
//     evict each other's lines before the next load comes back to them (4096
//     matrices of 32..2048 squared, b = 1..24: 1633 us against 1537); the copies
//     (memory to LDS) take whole rows' segments, consecutive lanes consecutive
//     chunks.
//   * A unit's words go to registers at once, and the next unit's copies are in
//     flight while they are decoded.  Two buffers in turn cost resident blocks:
//     1516 us, one buffer 1452.  No barrier: the buffer is the wave's own.
//   * 2^share waves can share a tile, its units dealt among them: each leaves its
//     rows' sums in part (LDS, 16 of the wave's own) for the caller to add.
// add: alpha times the sum of x.  w on a 16-byte boundary, of cap_bytes.
template <int B>
__device__ __forceinline__ void tiles(const uint32_t *__restrict__ w, uint64_t cap_bytes,
                                      int cols, int64_t row0, int64_t row_end, int wave,
                                      int waves, int64_t ntile, uint32_t flip,
                                      const uint8_t *xd, uint64_t add, uint8_t *buf,
                                      int64_t *__restrict__ y, int share, uint64_t *part) {
  typedef Unit<B> U;
  constexpr int L = (B + 7) / 8, D = kXDigits, CH = U::chunks;
  const int t0 = wave >> share, u0 = wave & ((1 << share) - 1);
  if (t0 >= ntile) return;
  // opaque: in a kernel that holds every width's code in a loop, what depends
  // on the lane alone would be computed for all of them before it (and spilled)
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const int n = lane & 15, h = lane >> 4;
  const int pitch = x_pitch(cols);
  const int nstep = (cols + kStep - 1) / kStep, nunit = (nstep + U::steps - 1) / U::steps;
  const uint8_t *xrow = xd + (n < D ? n : D) * pitch + 32 * h;
  const uint64_t weight = n < D ? 1ull << (8 * n) : n == D ? x_offset() : 0;

  // first bit of row r of tile t; rows past the end repeat the last one (their
  // results are not stored)
  auto row_bit = [&](int64_t t, int r) {
    int64_t row = row0 + t * kTileRows + r;
    row = row < row_end ? row : row_end - 1;
    return (uint64_t)row * (uint64_t)cols * B;
  };
  // byte offsets of this lane's copies of the tile's first unit, from `base`
  uint32_t off[U::insts];
  uint64_t base = 0;
  auto enter = [&](int64_t t) {
    base = row_bit(t, 0) / 128 * 16;
#pragma unroll
    for (int i = 0; i < U::insts; ++i) {
      int q = i * 64 + lane;
      q = q < kTileRows * CH ? q : kTileRows * CH - 1;
      off[i] = (uint32_t)(row_bit(t, q / CH) / 128 * 16 - base) + 16 * (q % CH);
    }
  };
  auto stage = [&](int u) {
    // this wave's LDS reads of the buffer have returned
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    const uint64_t at = base + (uint64_t)u * (16 * B * U::steps), end = cap_bytes - 16;
    const uint64_t from = at < end ? at : end;
    // chunks wholly past the payload hold no field: read its end instead
    const uint32_t lim = end - from < 0xfffffff0u ? (uint32_t)(end - from) : 0xfffffff0u;
    const global_ptr<uint8_t> src = as_global((const uint8_t *)w) + from;
#pragma unroll
    for (int i = 0; i < U::insts; ++i) {
      const uint32_t o = off[i] < lim ? off[i] : lim;
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void *)(src + o),
          (__attribute__((address_space(3))) void *)(buf + i * 1024), 16, 0, 0);
    }
  };
  v4i acc[L];
#pragma unroll
  for (int i = 0; i < L; ++i) acc[i] = v4i{0, 0, 0, 0};
  auto finish = [&](int64_t t) {
    // lane (n, h) holds column n of rows 4h .. 4h + 3
    uint64_t mine = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      uint64_t v = 0;
#pragma unroll
      for (int i = 0; i < L; ++i) v += (uint64_t)(int64_t)acc[i][r] << (8 * i);
      v *= weight;
      v = dpp_add64<0xB1>(v);  // sum over the 16 columns: quads,
      v = dpp_add64<0x4E>(v);
      v = dpp_add64<0x141>(v);  // then the half-row and row mirrors
      v = dpp_add64<0x140>(v);
      mine = n == r ? v : mine;
    }
#pragma unroll
    for (int i = 0; i < L; ++i) acc[i] = v4i{0, 0, 0, 0};
    const int64_t r = row0 + t * kTileRows + 4 * h + n;
    if (share) {
      if (n < 4) part[4 * h + n] = mine;
    } else if (n < 4 && r < row_end) {
      y[r] = (int64_t)(mine + add);
    }
  };

  int64_t t = t0, ts = t0;  // tile being decoded, tile being copied
  int u = u0;
  if (u0 >= nunit) {  // a narrow tile shared by more waves than it has units
    if (n < 4) part[4 * h + n] = 0;
    return;
  }
  enter(ts);
  stage(u0);
  // this lane's row of tile t: its funnel shift and its first word in a unit
  int sh = 0, word = 0;
  auto place = [&]() {
    const uint64_t bit = row_bit(t, n);
    sh = (int)(bit & 31u);
    word = n * CH * 4 + (int)((bit & 127u) >> 5) + h * B;
  };
  place();
  for (;;) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this unit's copies
    uint32_t ww[U::steps][B + 1];
    const uint32_t *aw = reinterpret_cast<const uint32_t *>(buf);
#pragma unroll
    for (int q = 0; q < U::steps; ++q)
#pragma unroll
      for (int k = 0; k <= B; ++k) ww[q][k] = aw[word + q * 4 * B + k];
    // the next unit's copies, while this one is decoded
    int un = u + (1 << share);
    if (un >= nunit) {
      un = u0;
      ts += waves >> share;
      if (ts < ntile) enter(ts);
    }
    const bool more = ts < ntile;
    if (more) stage(un);
#pragma unroll
    for (int q = 0; q < U::steps; ++q) {
      const int st = u * U::steps + q;
      if (U::steps == 1 || st < nstep) {  // the same for the wave
        const v4i b0 = *reinterpret_cast<const v4i *>(xrow + st * kStep);
        const v4i b1 = *reinterpret_cast<const v4i *>(xrow + st * kStep + 16);
#pragma unroll
        for (int k = 0; k < B; ++k)
          ww[q][k] = __builtin_amdgcn_alignbit(ww[q][k + 1], ww[q][k], sh);
        uint32_t o[L][8];
        tile_digits<B>(ww[q], flip, o);
#pragma unroll
        for (int i = 0; i < L; ++i) {
          const v4i a0 = {(int)o[i][0], (int)o[i][1], (int)o[i][2], (int)o[i][3]};
          const v4i a1 = {(int)o[i][4], (int)o[i][5], (int)o[i][6], (int)o[i][7]};
          acc[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a0, b0, acc[i], 0, 0, 0);
          acc[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a1, b1, acc[i], 0, 0, 0);
        }
      }
    }
    if (un == u0) finish(t);
    if (!more) break;
    if (ts != t) {
      t = ts;
      place();
    }
    u = un;
  }
}

}  // namespace mt
}  // namespace ccm
