// C = A B on matrix cores for packed operands of any width: the operands'
// values split into signed base-256 digits ("limbs"), every pair of limbs
// multiplied with v_mfma_i32_32x32x32_i8 in exact int32, the pairs combined
// in 64 bits (or 32 when every entry of C fits int32) as they are stored.
//
// Digits.  A field of b bits has L = ceil(b / 8) bytes u_i.  Digit i < L - 1
// is u_i - 128 (one XOR of the byte with 0x80); the top digit is the
// sign-extended top byte of a signed field, the byte itself of an unsigned
// one with at most 7 bits in it, and u_(L-1) - 128 when all 8 are in use.  So
// a = alpha + sum d_i 256^i with a constant alpha of the width, and
//   sum_k a b = sum_ij 256^(i+j) sum_k d_i e_j + alpha sum_k b + beta sum_k (a - alpha):
// the last two terms are one number per column and one per row of C, computed
// while the operands are decoded.  Digits are in [-128, 127], so a sum over
// K < 2^17 products stays inside int32.
//
// Layout of the decoded operands: K contiguous, zero-padded to a multiple of
// 128 (the K step); the L rows of digits of 32 matrix rows follow each other
// (row 32 g + r, limb i at stacked row (g L + i) 32 + r), so that the 32-row
// accumulator blocks of one wave hold every limb pair of its outputs and the
// combination never leaves the wave's registers.  The kernel is then the same
// GEMM over (L_A M) x (L_B N) stacked rows, whatever the limb counts.
//
// Bound by the matrix cores' issue (one limb each side: 468-480 us at 8192^3).
// Against the int64 vector path (us for the whole product, plan and pack):
// 12 x 10 bits, 1500 x 2000 x 1801: 79 against 539 (kernel 38-42).
#pragma once

#include <limits>
#include <type_traits>

#include "ccm_internal.hpp"
#include "group_codec.hpp"

namespace ccm {
namespace limb {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kBK = 128;  // K bytes per step (= LDS row)

// Digits of one operand: L limbs in chunks of at most `chunk` (a chunk is an
// array of its own; more than one only when the limb pairs of a product do
// not fit one wave's accumulators).
struct Limbs {
  int n;      // limbs in all
  int chunk;  // limbs per chunk (the last may have fewer)
};

__host__ __device__ inline int limbs_of(int bits) { return (bits + 7) / 8; }

// alpha: what the digits of a field leave out
__host__ __device__ inline uint64_t digit_offset(int bits, int sgn) {
  const int L = limbs_of(bits);
  uint64_t a = 0;
  for (int i = 0; i + 1 < L; ++i) a += 128ull << (8 * i);
  if (!sgn && bits % 8 == 0) a += 128ull << (8 * (L - 1));
  return a;
}

// Byte j of four 32-bit values as one word (value q in byte q).
template <int J>
__device__ __forceinline__ uint32_t bytes4(const uint32_t *v) {
  constexpr uint32_t sel = 0x0c0c0000u | ((uint32_t)(J + 4) << 8) | (uint32_t)J;
  const uint32_t lo = __builtin_amdgcn_perm(v[1], v[0], sel);
  const uint32_t hi = __builtin_amdgcn_perm(v[3], v[2], sel);
  return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}

// XOR that turns four top bytes (i == L - 1) or lower bytes into digits.
__device__ __forceinline__ uint32_t digit_flip(int bits, int sgn, int i, int L) {
  return i < L - 1 || (!sgn && bits % 8 == 0) ? 0x80808080u : 0u;
}

// The digits of 32 consecutive fields of B <= 32 bits, their words aligned:
// o[i][q] = digit i of fields 4q..4q+3.
template <int B>
__device__ __forceinline__ void words_digits(const uint32_t *ww, int sgn,
                                             uint32_t (&o)[(B + 7) / 8][8]) {
  constexpr int L = (B + 7) / 8;
  uint32_t v[32];
  if (sgn) {
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = codec::field32<B, true>(ww, i);
  } else {
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = codec::field32<B, false>(ww, i);
  }
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    o[0][q] = bytes4<0>(v + 4 * q) ^ digit_flip(B, sgn, 0, L);
    if constexpr (L > 1) o[1][q] = bytes4<1>(v + 4 * q) ^ digit_flip(B, sgn, 1, L);
    if constexpr (L > 2) o[2][q] = bytes4<2>(v + 4 * q) ^ digit_flip(B, sgn, 2, L);
    if constexpr (L > 3) o[3][q] = bytes4<3>(v + 4 * q) ^ digit_flip(B, sgn, 3, L);
  }
}

// Sum of the four signed bytes of a word, added to acc.
__device__ __forceinline__ int sum4(uint32_t w, int acc) {
  return __builtin_amdgcn_sdot4((int)w, 0x01010101, acc, false);
}

// 16-byte chunk c of tile row r sits at chunk position c ^ swz(r) of its
// 128-byte LDS row, so the MFMA operand reads (lanes 0-31 rows r..r+31 at one
// chunk, lanes 32-63 at the next) are conflict-free whether the LDS serves 8
// lanes of 16 bytes per cycle from 32 banks (8 consecutive rows take
// distinct positions) or 16 lanes from 64 banks (rows of equal parity among
// 16 take distinct positions); the bank-conflict counter reads 0.
__device__ __forceinline__ int swz(int r) { return (r ^ (r >> 3)) & 7; }

template <int FM, int FN>
__device__ __forceinline__ void mfma_slice(const v4i (&a)[FM], const v4i (&b)[FN],
                                           v16i (&acc)[FM][FN]) {
#pragma unroll
  for (int ta = 0; ta < FM; ++ta)
#pragma unroll
    for (int tb = 0; tb < FN; ++tb)
      acc[ta][tb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[ta], b[tb], acc[ta][tb], 0, 0, 0);
}

constexpr int kGroupM = 4;  // tile rows per group of the block order

// What a launch computes besides the digit products.
struct GemmArgs {
  const int8_t *A, *Bt;          // stacked digit rows of one chunk of A and of B
  int64_t arows, brows;          // stacked rows of each
  int64_t M, N, ldk;             // C is M x N; row pitch of the digits
  void *C;                       // dense C
  const int64_t *radd, *cadd;    // per row / column addends (null: none)
  int shift;                     // 8 (first limb of A's chunk + first of B's)
  int accumulate;                // add to C instead of storing
  RangeSink sink;                // exact range of C (null slots: not the last pass)
};

//   * Block = WGM x WGN waves; each wave owns FM x FN MFMA blocks of 32 x 32
//     stacked outputs (FM a multiple of LA, FN of LB), so FM + FN LDS reads of
//     16 bytes feed FM FN MFMAs.
//   * K steps of 128: the A and B tiles are copied into LDS with
//     memory-to-LDS loads (global_load_lds_dwordx4: each wave instruction
//     fills 8 rows, a lane's source chunk chosen so the row lands swizzled),
//     into the other of two buffers while the MFMAs consume this one.  Rows
//     past the end copy the last row (their outputs are not stored).
//   * One barrier per step, at its end, once the lane's copies of the next
//     step have landed (its LDS reads of this step have returned by then:
//     the barrier also waits for them, as it must: the buffer just read is
//     refilled right after it).
//   * The operands of each 32-deep slice of K are read one slice ahead into
//     a second register set, one LDS read issued after each MFMA; slice 0 of
//     a step is read after the barrier that completes its buffer.
//   * CORR: per-row and per-column addends (digit offsets).
template <int LA, int LB, int FM, int FN, int WGM, int WGN, typename OT, bool CORR>
__global__ __launch_bounds__(64 * WGM * WGN) void k_gemm_limb(GemmArgs p) {
  static_assert(FM % LA == 0 && FN % LB == 0, "a wave holds every limb pair of its outputs");
  constexpr int BM = 32 * FM * WGM, BN = 32 * FN * WGN;  // stacked tile
  constexpr int kWaves = WGM * WGN;
  constexpr size_t kTileBytes = (size_t)(BM + BN) * kBK;
  extern __shared__ __align__(16) int8_t gemm_lds[];
  const int64_t M = p.M, N = p.N, ldk = p.ldk;
  // Tile of this block.  Tiles are taken in groups of kGroupM tile rows
  // (consecutive tiles walk down the group, then across), and when the tile
  // count is a multiple of 8 each XCD (blocks are dealt to the 8 XCDs in
  // turn) gets one contiguous run of that order: the 32 blocks an XCD runs at
  // once then share 4 A panels and 8 B panels, whose K slices its L2 holds.
  const int64_t gx = (N + BN / LB - 1) / (BN / LB), gy = (M + BM / LA - 1) / (BM / LA);
  const int64_t ntile = gx * gy;
  int64_t tix = blockIdx.x;
  if (ntile % 8 == 0) tix = (tix % 8) * (ntile / 8) + tix / 8;
  const int64_t gsz_full = (int64_t)kGroupM * gx;
  const int64_t first_m = tix / gsz_full * kGroupM;
  const int64_t gsz = gy - first_m < kGroupM ? gy - first_m : kGroupM;
  const int64_t tm = first_m + (tix % gsz_full) % gsz, tn = (tix % gsz_full) / gsz;
  const int64_t s0 = tm * BM, t0 = tn * BN;  // first stacked rows of the tile
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;

  // the copy of one K step: BM + BN rows of 128 bytes, 8 rows per wave
  // instruction; instruction I: the tile's rows 8 I .. + 7 (A's first)
  constexpr int kRowsPerInst = 64 * 16 / kBK;
  static_assert((BM + BN) / kRowsPerInst % kWaves == 0 && BM % kRowsPerInst == 0, "copy split");
  constexpr int kInstPerWave = (BM + BN) / kRowsPerInst / kWaves;
  constexpr int kChunks = kBK / 16;
  const int lrow = lane / kChunks, lpos = lane % kChunks;
  auto stage = [&](int64_t k0, int buf) {
#pragma unroll
    for (int q = 0; q < kInstPerWave; ++q) {
      const int I = wave * kInstPerWave + q;
      const int opnd = I >= BM / kRowsPerInst ? 1 : 0;
      const int rb = kRowsPerInst * I - (opnd ? BM : 0);
      const int r = rb + lrow;
      const int64_t lim = opnd ? p.brows : p.arows;
      int64_t gr = (opnd ? t0 : s0) + r;
      gr = gr < lim ? gr : lim - 1;
      const int c = lpos ^ swz(r);
      const int8_t *src = (opnd ? p.Bt : p.A) + gr * ldk + k0 + 16 * c;
      int8_t *dst = gemm_lds + (size_t)buf * kTileBytes + (size_t)I * kRowsPerInst * kBK;
      __builtin_amdgcn_global_load_lds((const void *)src,
                                       (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
    }
  };
  // LDS offsets of this lane's operand rows and their swizzle
  int aoff[FM], boff[FN], asw[FM], bsw[FN];
#pragma unroll
  for (int t = 0; t < FM; ++t) {
    const int r = (wm * FM + t) * 32 + (lane & 31);
    aoff[t] = r * kBK;
    asw[t] = swz(r);
  }
#pragma unroll
  for (int t = 0; t < FN; ++t) {
    const int r = (wn * FN + t) * 32 + (lane & 31);
    boff[t] = BM * kBK + r * kBK;
    bsw[t] = swz(r);
  }
  // lanes 0-31 take bytes 0-15 of the slice's 32 K values, lanes 32-63 bytes
  // 16-31, for both operands
  auto fetch = [&](int buf, int kk, v4i(&a)[FM], v4i(&b)[FN]) {
    const int8_t *base = gemm_lds + (size_t)buf * kTileBytes;
    const int c = kk / 16 + (lane >> 5);
#pragma unroll
    for (int t = 0; t < FM; ++t)
      a[t] = *reinterpret_cast<const v4i *>(base + aoff[t] + 16 * (c ^ asw[t]));
#pragma unroll
    for (int t = 0; t < FN; ++t)
      b[t] = *reinterpret_cast<const v4i *>(base + boff[t] + 16 * (c ^ bsw[t]));
  };

  v16i acc[FM][FN];
#pragma unroll
  for (int a = 0; a < FM; ++a)
#pragma unroll
    for (int b = 0; b < FN; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0;

  const int64_t nk = ldk / kBK;
  stage(0, 0);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  // two operand sets: the reads of slice s + 1 are in flight during the
  // MFMAs of slice s (within a step; slice 0 of the next step is read after
  // the barrier, once its buffer is complete)
  v4i a0[FM], b0[FN], a1[FM], b1[FN];
  fetch(0, 0, a0, b0);
  for (int64_t kc = 0; kc < nk; ++kc) {
    const int cur = (int)(kc & 1);
    if (kc + 1 < nk) stage((kc + 1) * kBK, cur ^ 1);  // in flight during the MFMAs
#pragma unroll
    for (int s = 0; s < kBK / 32; ++s) {
      if (s % 2 == 0) {
        if (s + 1 < kBK / 32) fetch(cur, 32 * (s + 1), a1, b1);
        mfma_slice<FM, FN>(a0, b0, acc);
      } else {
        if (s + 1 < kBK / 32) fetch(cur, 32 * (s + 1), a0, b0);
        mfma_slice<FM, FN>(a1, b1, acc);
      }
      if (s + 1 < kBK / 32) {
        // one LDS read after each of the first MFMAs, then the rest
#pragma unroll
        for (int q = 0; q < FM + FN; ++q) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // an MFMA
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // an LDS read
        }
        if constexpr (FM * FN > FM + FN)
          __builtin_amdgcn_sched_group_barrier(0x008, FM * FN - (FM + FN), 0);
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this lane's copies of the next step
    __syncthreads();  // everyone's copies have landed and this buffer is read
    if (kc + 1 < nk) fetch(cur ^ 1, 0, a0, b0);
  }

  // 32x32 accumulator layout: lane l, register r -> column l%32,
  // row 8*(r/4) + 4*(l/32) + r%4.  Row offsets are uniform multiples of N.
  constexpr int GM = FM / LA, GN = FN / LB;  // 32-row groups of C per wave
  typedef typename std::conditional<sizeof(OT) == 4, uint32_t, uint64_t>::type UT;
  OT lo = std::numeric_limits<OT>::max(), hi = std::numeric_limits<OT>::min();
  const int64_t rbase = tm * (BM / LA) + wm * GM * 32 + 4 * (lane >> 5);
  const int64_t cbase = tn * (BN / LB) + wn * GN * 32 + (lane & 31);
  OT *cp = (OT *)p.C + rbase * N + cbase;
  UT cadd[GN];
  if constexpr (CORR) {
#pragma unroll
    for (int h = 0; h < GN; ++h)
      cadd[h] = p.cadd && cbase + 32 * h < N ? (UT)(uint64_t)p.cadd[cbase + 32 * h] : UT(0);
  }
#pragma unroll
  for (int g = 0; g < GM; ++g)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int ro = g * 32 + 8 * (r / 4) + (r % 4);
      OT *rowp = cp + (int64_t)ro * N;
      const bool rok = rbase + ro < M;
      UT radd = 0;
      if constexpr (CORR) {
        if (p.radd && rok) radd = (UT)(uint64_t)p.radd[rbase + ro];
      }
#pragma unroll
      for (int h = 0; h < GN; ++h) {
        UT v = 0;
#pragma unroll
        for (int i = 0; i < LA; ++i)
#pragma unroll
          for (int j = 0; j < LB; ++j)
            if (8 * (i + j) < 8 * (int)sizeof(OT))
              v += (UT)(int64_t)acc[g * LA + i][h * LB + j][r] << (8 * (i + j));
        if constexpr (CORR) {
          v = (UT)(v << p.shift) + radd + cadd[h];
        }
        if (rok && cbase + 32 * h < N) {
          if constexpr (CORR && sizeof(OT) == 8) {
            if (p.accumulate) v += (UT)rowp[32 * h];
          }
          const OT o = (OT)v;
          rowp[32 * h] = o;
          lo = o < lo ? o : lo;
          hi = o > hi ? o : hi;
        }
      }
      __builtin_amdgcn_sched_barrier(0);  // one row at a time: no copies of all accumulators
    }
  if (p.sink.slot) block_range_commit((int64_t)lo, (int64_t)hi, 0, p.sink);
}

// Rows and columns of C per block of a pass over la x lb limbs.
constexpr int tile_rows(int la) { return la == 1 ? 256 : la == 2 ? 128 : 64; }
constexpr int tile_cols(int la, int lb) { return lb == 1 ? 256 : lb == 2 || la == 3 ? 128 : 64; }

template <int LA, int LB, int FM, int FN, int WGM, int WGN, typename OT, bool CORR>
hipError_t launch_tile(const GemmArgs &p, hipStream_t s) {
  constexpr int BM = 32 * FM * WGM, BN = 32 * FN * WGN;
  static_assert(BM / LA == tile_rows(LA) && BN / LB == tile_cols(LA, LB), "tile");
  constexpr size_t lds = 2u * (size_t)(BM + BN) * kBK;
  const int64_t ntile = ((p.N + BN / LB - 1) / (BN / LB)) * ((p.M + BM / LA - 1) / (BM / LA));
  if (ntile > 0x7fffffffll) return hipErrorInvalidValue;
  auto kern = k_gemm_limb<LA, LB, FM, FN, WGM, WGN, OT, CORR>;
  static const hipError_t attr =
      hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  (void)attr;
  kern<<<(unsigned)ntile, 64 * WGM * WGN, lds, s>>>(p);
  return hipGetLastError();
}

// C = A B for a narrow right operand of one digit without offset
// (gemm_skinny.hpp).
constexpr int kSkRows = 128;  // rows of A per block
// 16-byte chunks copied per row and step: the 16 B bytes of 128 fields, up to
// 15 before them and the word after the last, rounded up to odd.
constexpr int sk_chunks(int B) { return (B + 2) | 1; }
constexpr int sk_insts(int B) { return (32 * sk_chunks(B) + 63) / 64; }
constexpr int sk_stage(int B, int NB) { return 4 * sk_insts(B) * 1024 + NB * 32 * kBK; }
struct SkinnyArgs {
  const uint32_t *aw;
  uint64_t cap_bytes;
  int sgn;
  int64_t M, K, N, ldk;
  const int8_t *Bt;  // N digit rows
  int64_t kper;
  int splits;
  int64_t *part;        // splits x M x N partial sums (splits > 1)
  uint64_t alpha;       // what A's digits leave out
  void *C;
  int out32;
  RangeSink sink;
};
hipError_t launch_skinny_1(const SkinnyArgs &p, int abits, int nb, hipStream_t s);
hipError_t launch_skinny_2(const SkinnyArgs &p, int abits, int nb, hipStream_t s);
hipError_t launch_skinny_3(const SkinnyArgs &p, int abits, int nb, hipStream_t s);
hipError_t launch_skinny_4(const SkinnyArgs &p, int abits, int nb, hipStream_t s);
// ... of at most 64 columns (gemm_narrow.hpp); the digits of B in chunk tiles:
// byte offset of digits k .. k + 15 (k a multiple of 16) of column n, for `blocks`
// blocks of 16 columns.  1 KB per K step, block and MFMA of the step (k / 16 % 2),
// then 16 bytes per lane (16 (k / 32 % 4) + n % 16).
__host__ __device__ inline int64_t chunk_tile(int64_t n, int64_t k, int blocks) {
  return ((k / kBK * blocks + n / 16) * 2 + k / 16 % 2) * 1024 + (k / 32 % 4 * 16 + n % 16) * 16;
}
hipError_t launch_narrow_1(const SkinnyArgs &p, int abits, int waves, hipStream_t s);
hipError_t launch_narrow_2(const SkinnyArgs &p, int abits, int waves, hipStream_t s);
hipError_t launch_narrow_3(const SkinnyArgs &p, int abits, int waves, hipStream_t s);
hipError_t launch_narrow_4(const SkinnyArgs &p, int abits, int waves, hipStream_t s);

// One pass over a chunk of la limbs of A and lb of B (la, lb <= 3, or 4 with
// at most 2 on the other side); OT int32 (out32) or int64.
hipError_t launch_pass(const GemmArgs &p, int la, int lb, int out32, hipStream_t s);
hipError_t launch_pass_a1(const GemmArgs &p, int lb, int out32, hipStream_t s);
hipError_t launch_pass_a2(const GemmArgs &p, int lb, int out32, hipStream_t s);
hipError_t launch_pass_a3(const GemmArgs &p, int lb, int out32, hipStream_t s);
hipError_t launch_pass_a4(const GemmArgs &p, int lb, int out32, hipStream_t s);

}  // namespace limb
}  // namespace ccm
