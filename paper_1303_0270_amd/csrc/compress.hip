// Compression in one pass over a large dense matrix: packed at a width guessed
// from a sample while the exact range is reduced.
//
// The width of a matrix is known only once its range is, so packing reads the
// dense values a second time; both passes run at the rate of memory.  A sample
// of the values almost always has the width of them all (the extremes of
// 2^18 values against those of all of them: the same power of two unless the
// larger ones are very rare), so the packing pass runs at the sample's width
// and reduces the exact range on the way; when that range has the same width,
// the payload is final.  A block that meets a value outside the guess stops
// the packing: later blocks only reduce the range, so a wrong guess costs
// about the sample and what had been written, not a second pass.
// Measured, 16384 x 16384 int64 at 12 bits (2.55 GB in and out), us a call: range
// and pack 870 (406 + 454), here 502; with one value past the guess 1 / 50 /
// 99.9 % into the matrix 855 / 908 / 960.
//
// A block stages 256 groups through LDS as their low words (fields of at most
// 31 bits, or int32 input: half the LDS of int64 values, so 16 waves a CU
// keep 512 KB of loads in flight), lane g encodes group g at the compile-time
// width, and the block's run of words leaves with 16-byte nontemporal stores.
#include <type_traits>

#include "ccm_internal.hpp"
#include "group_codec.hpp"

namespace ccm {
namespace {

constexpr int kSampleBlocks = 512, kSampleThreads = 256;

// The range of a sample: each block takes the 16-byte pieces of one run, the
// runs spread evenly over the matrix.
template <typename T>
__global__ __launch_bounds__(kSampleThreads) void k_sample_range(const T *__restrict__ d,
                                                                 uint64_t n, RangeSink sink) {
  constexpr int PER = 16 / sizeof(T);
  const uint64_t run = (uint64_t)kSampleThreads * PER;
  const uint64_t at = n > run ? (n - run) / (kSampleBlocks - 1) * blockIdx.x : 0;
  int64_t lo = INT64_MAX, hi = INT64_MIN;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const uint64_t e = at + (uint64_t)u * kSampleThreads + threadIdx.x;
    if (e < n) {
      const int64_t x = (int64_t)d[e];
      lo = x < lo ? x : lo;
      hi = x > hi ? x : hi;
    }
  }
  block_range_commit(lo, hi, 0, sink);
}

template <int B, typename T>
constexpr bool low_words() {
  return sizeof(T) == 4 || B <= 31;
}
template <int B, typename T>
constexpr int pack_threads() {
  return low_words<B, T>() ? 256 : 128;
}

// Packs at B bits and folds the exact range; [glo, ghi] is what fits the guess.
// sink.full[1] is the stop word, and the slot's flag tells the host of it.
template <int B, typename T>
__global__ __launch_bounds__((pack_threads<B, T>())) void k_compress_range(
    const T *__restrict__ d, uint64_t n, int64_t glo, int64_t ghi, uint32_t *__restrict__ out,
    uint64_t cap32, RangeSink sink, int aligned16) {
  constexpr bool LOW = low_words<B, T>();
  constexpr int NT = pack_threads<B, T>();
  typedef typename std::conditional<LOW, uint32_t, int64_t>::type V;
  constexpr int PER = 16 / sizeof(T), NLOAD = kGroup / PER, kPitch = kGroup + 1;
  constexpr size_t kTile = sizeof(V) * NT * kPitch, kOut = 4 * (size_t)NT * B;
  __shared__ __align__(16) unsigned char lds[kTile > kOut ? kTile : kOut];
  __shared__ int64_t s_lo[NT / 64], s_hi[NT / 64];
  __shared__ uint32_t s_stop;
  V *tile = reinterpret_cast<V *>(lds);
  const int tid = threadIdx.x;
  const uint64_t e0 = (uint64_t)blockIdx.x * NT * kGroup;
  int64_t lo = INT64_MAX, hi = INT64_MIN;
  if (tid == 0) s_stop = *(volatile uint32_t *)(sink.full + 1);
  if (aligned16 && e0 + (uint64_t)NT * kGroup <= n) {
    const uint4 *src = reinterpret_cast<const uint4 *>(d + e0);
    uint4 r[NLOAD];
#pragma unroll
    for (int j = 0; j < NLOAD; ++j) r[j] = src[tid + j * NT];
    if constexpr (sizeof(T) == 4 || LOW) {
      // 32-bit extremes of the low words; they are the values' own while every
      // high word is the low one's sign
      int32_t mn = INT32_MAX, mx = INT32_MIN;
      uint32_t odd = 0;
#pragma unroll
      for (int j = 0; j < NLOAD; ++j) {
        const int q = (tid + j * NT) * PER;
        const uint32_t w[4] = {r[j].x, r[j].y, r[j].z, r[j].w};
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          const int32_t x = (int32_t)w[u * (4 / PER)];
          if constexpr (sizeof(T) == 8) odd |= w[2 * u + 1] ^ (uint32_t)(x >> 31);
          mn = x < mn ? x : mn;
          mx = x > mx ? x : mx;
          tile[q + u + (q >> 5)] = (V)(uint32_t)x;
        }
      }
      lo = mn;
      hi = mx;
      if (sizeof(T) == 8 && odd) {
        lo = INT64_MAX;
        hi = INT64_MIN;
#pragma unroll
        for (int j = 0; j < NLOAD; ++j) {
          const int64_t a = (int64_t)(((uint64_t)r[j].y << 32) | r[j].x);
          const int64_t b = (int64_t)(((uint64_t)r[j].w << 32) | r[j].z);
          lo = a < lo ? a : lo;
          hi = a > hi ? a : hi;
          lo = b < lo ? b : lo;
          hi = b > hi ? b : hi;
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < NLOAD; ++j) {
        const int q = (tid + j * NT) * PER;
        const int64_t a = (int64_t)(((uint64_t)r[j].y << 32) | r[j].x);
        const int64_t b = (int64_t)(((uint64_t)r[j].w << 32) | r[j].z);
        lo = a < lo ? a : lo;
        hi = a > hi ? a : hi;
        lo = b < lo ? b : lo;
        hi = b > hi ? b : hi;
        tile[q + (q >> 5)] = (V)a;
        tile[q + 1 + (q >> 5)] = (V)b;
      }
    }
  } else {
    for (int q = tid; q < NT * kGroup; q += NT) {
      const uint64_t e = e0 + q;
      int64_t x = 0;
      if (e < n) {
        x = (int64_t)d[e];
        lo = x < lo ? x : lo;
        hi = x > hi ? x : hi;
      }
      tile[q + (q >> 5)] = (V)x;
    }
  }
  lo = wave_min(lo);
  hi = wave_max(hi);
  if ((tid & 63) == 0) {
    s_lo[tid >> 6] = lo;
    s_hi[tid >> 6] = hi;
  }
  __syncthreads();
  if (tid == 0) {
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) {
      lo = s_lo[w] < lo ? s_lo[w] : lo;
      hi = s_hi[w] > hi ? s_hi[w] : hi;
    }
    // as in the add's packing grid: an atomic only where the extreme beats what
    // the slot holds (a slot only narrows)
    RangeSlot *r = sink.slot + kRangeStride * (blockIdx.x % kRangeSpread);
    const int64_t seen_lo = __hip_atomic_load(&r->vmin, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int64_t seen_hi = __hip_atomic_load(&r->vmax, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (lo < seen_lo) atomicMin((long long *)&r->vmin, (long long)lo);
    if (hi > seen_hi) atomicMax((long long *)&r->vmax, (long long)hi);
    if (lo <= hi && (lo < glo || hi > ghi)) {
      atomicOr(&r->flag, 1);
      atomicOr(sink.full + 1, 1u);
    }
  }
  if (s_stop) return;  // the same for the whole block
  V v[kGroup];
#pragma unroll
  for (int i = 0; i < kGroup; ++i) v[i] = tile[tid * kPitch + i];
  __syncthreads();
  uint32_t *s_out = reinterpret_cast<uint32_t *>(lds);
  if constexpr (LOW && B <= 32)
    codec::encode32<B>(reinterpret_cast<const uint32_t *>(v), s_out + tid * B, (uint64_t)B);
  else if constexpr (!LOW)
    codec::encode<B>(reinterpret_cast<const int64_t *>(v), s_out + tid * B, (uint64_t)B);
  __syncthreads();
  store_block_run(s_out, B, out, cap32);
}

template <typename T>
hipError_t launch_one(const T *d, uint64_t n, int bits, int64_t glo, int64_t ghi, uint32_t *out,
                      uint64_t cap32, RangeSink sink, hipStream_t s) {
  const uint64_t ngroups = (cap32 + bits - 1) / bits;
  const int al = ((uintptr_t)d % 16) == 0;
  switch (bits) {
#define CCM_COMPRESS_RANGE(b)                                                                     \
  case b: {                                                                                       \
    if constexpr (b <= 32 || sizeof(T) == 8) {                                                    \
      constexpr int nt = pack_threads<b, T>();                                                    \
      const uint64_t grid = (ngroups + nt - 1) / nt;                                              \
      if (grid > 0x7fffffffull) return hipErrorInvalidValue;                                      \
      k_compress_range<b, T><<<(unsigned)grid, nt, 0, s>>>(d, n, glo, ghi, out, cap32, sink, al); \
    } else {                                                                                      \
      return hipErrorInvalidValue;                                                                \
    }                                                                                             \
    break;                                                                                        \
  }
    CCM_WIDTH_CASES(CCM_COMPRESS_RANGE)
#undef CCM_COMPRESS_RANGE
    default: return hipErrorInvalidValue;
  }
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : launch_range_publish(sink, s);
}

}  // namespace

hipError_t launch_sample_range(const void *dense, int dtype, uint64_t n, RangeSink sink,
                               hipStream_t s) {
  if (dtype == CCM_I64)
    k_sample_range<int64_t>
        <<<kSampleBlocks, kSampleThreads, 0, s>>>((const int64_t *)dense, n, sink);
  else
    k_sample_range<int32_t>
        <<<kSampleBlocks, kSampleThreads, 0, s>>>((const int32_t *)dense, n, sink);
  return hipGetLastError();
}

hipError_t launch_compress_range(const void *dense, int dtype, uint64_t n, int bits, int64_t glo,
                                 int64_t ghi, uint32_t *out, uint64_t cap32, RangeSink sink,
                                 hipStream_t s) {
  if (dtype == CCM_I64)
    return launch_one<int64_t>((const int64_t *)dense, n, bits, glo, ghi, out, cap32, sink, s);
  return launch_one<int32_t>((const int32_t *)dense, n, bits, glo, ghi, out, cap32, sink, s);
}

}  // namespace ccm
