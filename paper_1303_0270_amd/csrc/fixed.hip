// Floats in fixed point (the Conclusion allows floats if some precision is
// given up): the quantization that turns a float matrix into the integer
// matrix Method 1 packs, the exact largest magnitude that picks its scale,
// and the conversion of integer results back to floats (gfx950).
//
//   q = round-half-to-even(v * 2^f): v_ldexp_f64 scales exactly (or leaves
//   the double range: then |v 2^f| is far beyond 2^62, or below 2^-1022,
//   where the rounding gives 0 either way), v_rndne_f64 rounds half to even.
//   Back: int64 -> double rounds half to even (one rounding: the high half
//   scaled by 2^32 plus the exact low half), ldexp by -f, and for float32 one
//   more rounding (v_cvt_f32_f64, round to nearest even).
#include "ccm_internal.hpp"
#include "group_codec.hpp"

#include <cmath>
#include <limits>
#include <type_traits>

namespace ccm {
namespace {

constexpr int kFxThreads = 256;

// Integers that order like the values they came from (-0 below +0): negative
// NaNs sort below -infinity, the others above +infinity, so the extremes of
// the integers tell of any NaN or infinity.
__device__ __forceinline__ int64_t ordered(double v) {
  const int64_t b = __double_as_longlong(v);
  return b ^ ((b >> 63) & INT64_MAX);
}
__device__ __forceinline__ int32_t ordered(float v) {
  const int32_t b = __float_as_int(v);
  return b ^ ((b >> 31) & INT32_MAX);
}
__device__ __forceinline__ double unordered(int64_t o) {
  return __longlong_as_double(o ^ ((o >> 63) & INT64_MAX));
}
__device__ __forceinline__ double unordered(int32_t o) {
  return (double)__int_as_float(o ^ ((o >> 31) & INT32_MAX));
}
// the extremes of a type's integers as a double's
template <typename O>
__device__ __forceinline__ int64_t widened(O o) {
  if constexpr (sizeof(O) == 8)
    return o;
  else
    return ordered(unordered(o));
}
template <typename F>
struct OrderedOf {
  typedef int64_t type;
};
template <>
struct OrderedOf<float> {
  typedef int32_t type;
};

// Exact (min, max) of n floats as ordered integers; 16-byte loads, four in
// flight per lane.
template <typename F>
__global__ __launch_bounds__(kFxThreads) void k_float_range(const F *__restrict__ v, uint64_t n,
                                                            RangeSink sink, int aligned16) {
  typedef typename OrderedOf<F>::type O;
  constexpr int PER = 16 / sizeof(F), UNR = 4;
  O lo = std::numeric_limits<O>::max(), hi = std::numeric_limits<O>::min();
  auto fold = [&](F x) {
    const O o = ordered(x);
    lo = o < lo ? o : lo;
    hi = o > hi ? o : hi;
  };
  const uint64_t tid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  uint64_t done = 0;
  if (aligned16) {
    const uint64_t n16 = n / PER;
    const uint4 *p = reinterpret_cast<const uint4 *>(v);
    uint64_t i = tid;
    for (; i + (UNR - 1) * stride < n16; i += UNR * stride) {
      uint4 r[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) r[u] = p[i + u * stride];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const F *t = reinterpret_cast<const F *>(&r[u]);
#pragma unroll
        for (int q = 0; q < PER; ++q) fold(t[q]);
      }
    }
    for (; i < n16; i += stride) {
      const uint4 r = p[i];
      const F *t = reinterpret_cast<const F *>(&r);
#pragma unroll
      for (int q = 0; q < PER; ++q) fold(t[q]);
    }
    done = n16 * PER;
  }
  for (uint64_t e = done + tid; e < n; e += stride) fold(v[e]);
  const bool any = lo <= hi;
  block_range_commit(any ? widened(lo) : INT64_MAX, any ? widened(hi) : INT64_MIN, 0, sink);
}

// The range of a sample: each block takes one run, the runs spread evenly.
constexpr int kSampleBlocks = 512, kSamplePer = 4;
template <typename F>
__global__ __launch_bounds__(kFxThreads) void k_float_sample(const F *__restrict__ v, uint64_t n,
                                                             RangeSink sink) {
  typedef typename OrderedOf<F>::type O;
  const uint64_t run = (uint64_t)kFxThreads * kSamplePer;
  const uint64_t at = n > run ? (n - run) / (kSampleBlocks - 1) * blockIdx.x : 0;
  O lo = std::numeric_limits<O>::max(), hi = std::numeric_limits<O>::min();
#pragma unroll
  for (int u = 0; u < kSamplePer; ++u) {
    const uint64_t e = at + (uint64_t)u * kFxThreads + threadIdx.x;
    if (e < n) {
      const O o = ordered(v[e]);
      lo = o < lo ? o : lo;
      hi = o > hi ? o : hi;
    }
  }
  const bool any = lo <= hi;
  block_range_commit(any ? widened(lo) : INT64_MAX, any ? widened(hi) : INT64_MIN, 0, sink);
}

// q = RNE(v 2^f) with the range of q folded into slot.  A NaN or infinity
// sets the slot's flag; a |v 2^f| >= 2^62, or for int32 output a q outside
// int32, folds INT64_MAX into the maximum (every valid q is below 2^62 in
// magnitude).
// q may be null: the range and the checks only.  With a null sink the values
// were checked before and only q is written.
template <typename F, typename Q>
__global__ __launch_bounds__(kFxThreads) void k_quantize(const F *__restrict__ v, uint64_t n,
                                                         int f, Q *__restrict__ q,
                                                         RangeSink sink) {
  int64_t lo = INT64_MAX, hi = INT64_MIN;
  int bad = 0;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  auto one = [&](F x, uint64_t e) {
    const double d = (double)x;
    const double t = ldexp(d, f);
    int64_t r = 0;
    if (!isfinite(d)) {
      bad = 1;
    } else if (!(fabs(t) < 0x1p62)) {
      hi = INT64_MAX;
    } else {
      r = (int64_t)rint(t);
      if (sizeof(Q) == 4 && (r < INT32_MIN || r > INT32_MAX)) {
        hi = INT64_MAX;
        r = 0;
      } else {
        lo = r < lo ? r : lo;
        hi = r > hi ? r : hi;
      }
    }
    if (q) q[e] = (Q)r;
  };
  uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (; i + 3 * stride < n; i += 4 * stride) {
    F t[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) t[u] = v[i + u * stride];
#pragma unroll
    for (int u = 0; u < 4; ++u) one(t[u], i + u * stride);
  }
  for (; i < n; i += stride) one(v[i], i);
  if (sink.slot) block_range_commit(lo, hi, bad, sink);
}

template <typename F>
__global__ __launch_bounds__(kFxThreads) void k_dequantize(const int64_t *__restrict__ q,
                                                           uint64_t n, int f,
                                                           F *__restrict__ out) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (; i + 3 * stride < n; i += 4 * stride) {
    int64_t t[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) t[u] = q[i + u * stride];
#pragma unroll
    for (int u = 0; u < 4; ++u) out[i + u * stride] = (F)ldexp((double)t[u], -f);
  }
  for (; i < n; i += stride) out[i] = (F)ldexp((double)q[i], -f);
}

// Packs RNE(v 2^f) at `bits` straight from the floats: a block stages its
// 32 x 128 floats through LDS with 16-byte loads, then lane g quantizes group
// g's 32 values and encodes its b words (as the integer packing kernel does).
// The values were checked by the range pass before (finite, inside the
// width), so no test is repeated here.
constexpr int kFxTile = 128;
constexpr int kFxPad = kGroup + 1;

template <typename F>
__global__ __launch_bounds__(kFxTile) void k_compress_fx(const F *__restrict__ d, uint64_t n,
                                                         int f, int bits,
                                                         uint32_t *__restrict__ out,
                                                         uint64_t cap32, uint64_t ngroups,
                                                         int aligned16) {
  constexpr int PER = 16 / sizeof(F);
  constexpr int NLOAD = kFxTile * kGroup / (kFxTile * PER);
  // the input tile, reused for the block's packed words (up to 64 a group)
  constexpr size_t kBytes = sizeof(F) * kFxTile * kFxPad > 4 * (size_t)kFxTile * 64
                                ? sizeof(F) * kFxTile * kFxPad
                                : 4 * (size_t)kFxTile * 64;
  __shared__ __align__(16) unsigned char lds[kBytes];
  F *tile = reinterpret_cast<F *>(lds);
  const uint64_t g0 = (uint64_t)blockIdx.x * kFxTile;
  const uint64_t e0 = g0 * kGroup;
  if (aligned16 && e0 + (uint64_t)kFxTile * kGroup <= n) {
    const uint4 *src = reinterpret_cast<const uint4 *>(d + e0);
    uint4 r[NLOAD];
#pragma unroll
    for (int j = 0; j < NLOAD; ++j) r[j] = src[threadIdx.x + j * kFxTile];
#pragma unroll
    for (int j = 0; j < NLOAD; ++j) {
      const int q = (threadIdx.x + j * kFxTile) * PER;
      const F *t = reinterpret_cast<const F *>(&r[j]);
#pragma unroll
      for (int u = 0; u < PER; ++u) tile[q + u + (q >> 5)] = t[u];
    }
  } else {
    for (int q = threadIdx.x; q < kFxTile * kGroup; q += kFxTile) {
      const uint64_t e = e0 + q;
      tile[q + (q >> 5)] = e < n ? d[e] : F(0);
    }
  }
  __syncthreads();
  int64_t v[kGroup];
  const F *row = tile + threadIdx.x * kFxPad;
#pragma unroll
  for (int i = 0; i < kGroup; ++i) v[i] = (int64_t)rint(ldexp((double)row[i], f));
  // group g into LDS, then the block's contiguous run of words (as the
  // integer packing kernel)
  __syncthreads();
  uint32_t *s_out = reinterpret_cast<uint32_t *>(lds);
  codec::encode_rt(v, bits, s_out + threadIdx.x * bits, (uint64_t)bits);
  __syncthreads();
  store_block_run(s_out, bits, out, cap32);
  (void)ngroups;
}

// Packs RNE(v 2^f) at B bits while the exact range of v is reduced: the float
// form of the integers' one-pass packing (a width guessed from a sample; the
// stop word and the flag as there).  [qlo, qhi]: the q that fit B bits.  Bound
// by memory: 16384 x 8192 float32 to 13 bits (0.76 GB in and out) in 135 us,
// with 9 us of sample before it; the largest magnitude, the range of q and the
// packing took 119 + 123 + 119 us, each reading the floats again.
template <int B, typename F>
__global__ __launch_bounds__(B <= 31 ? 256 : 128) void k_compress_fx_range(
    const F *__restrict__ d, uint64_t n, int f, double qlo, double qhi,
    uint32_t *__restrict__ out, uint64_t cap32, RangeSink sink, int aligned16) {
  constexpr bool LOW = B <= 31;
  constexpr int NT = LOW ? 256 : 128;
  typedef typename std::conditional<LOW, int32_t, int64_t>::type V;
  typedef typename OrderedOf<F>::type O;
  constexpr int PER = 16 / sizeof(F), NLOAD = kGroup / PER, kPitch = kGroup + 1;
  constexpr size_t kTile = sizeof(V) * NT * kPitch, kOut = 4 * (size_t)NT * B;
  __shared__ __align__(16) unsigned char lds[kTile > kOut ? kTile : kOut];
  __shared__ int64_t s_lo[NT / 64], s_hi[NT / 64];
  __shared__ uint32_t s_stop;
  V *tile = reinterpret_cast<V *>(lds);
  const int tid = threadIdx.x;
  const uint64_t e0 = (uint64_t)blockIdx.x * NT * kGroup;
  O mn = std::numeric_limits<O>::max(), mx = std::numeric_limits<O>::min();
  auto put = [&](int q, F x) {
    const O o = ordered(x);
    mn = o < mn ? o : mn;
    mx = o > mx ? o : mx;
    tile[q + (q >> 5)] = (V)rint(ldexp((double)x, f));
  };
  if (tid == 0) s_stop = *(volatile uint32_t *)(sink.full + 1);
  if (aligned16 && e0 + (uint64_t)NT * kGroup <= n) {
    const uint4 *src = reinterpret_cast<const uint4 *>(d + e0);
    uint4 r[NLOAD];
#pragma unroll
    for (int j = 0; j < NLOAD; ++j) r[j] = src[tid + j * NT];
#pragma unroll
    for (int j = 0; j < NLOAD; ++j) {
      const F *t = reinterpret_cast<const F *>(&r[j]);
#pragma unroll
      for (int u = 0; u < PER; ++u) put((tid + j * NT) * PER + u, t[u]);
    }
  } else {
    for (int q = tid; q < NT * kGroup; q += NT) {
      if (e0 + q < n)
        put(q, d[e0 + q]);
      else
        tile[q + (q >> 5)] = 0;
    }
  }
  int64_t lo = mn <= mx ? widened(mn) : INT64_MAX, hi = mn <= mx ? widened(mx) : INT64_MIN;
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
    RangeSlot *r = sink.slot + kRangeStride * (blockIdx.x % kRangeSpread);
    const int64_t seen_lo = __hip_atomic_load(&r->vmin, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int64_t seen_hi = __hip_atomic_load(&r->vmax, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (lo < seen_lo) atomicMin((long long *)&r->vmin, (long long)lo);
    if (hi > seen_hi) atomicMax((long long *)&r->vmax, (long long)hi);
    // a NaN fails both comparisons
    if (lo <= hi && !(rint(ldexp(unordered(lo), f)) >= qlo && rint(ldexp(unordered(hi), f)) <= qhi)) {
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
  if constexpr (LOW)
    codec::encode32<B>(reinterpret_cast<const uint32_t *>(v), s_out + tid * B, (uint64_t)B);
  else
    codec::encode<B>(v, s_out + tid * B, (uint64_t)B);
  __syncthreads();
  store_block_run(s_out, B, out, cap32);
}

// out = q 2^-f straight from the packed fields (through int64 in memory the same
// conversion moved 16 bytes an element more: 16384 x 8192 at 13 bits to float32
// in 501 us, 180 of them decoding; here 107 us).
template <int B, typename F>
__global__ __launch_bounds__(B <= 31 ? 256 : 128) void k_decompress_fx(
    const uint32_t *__restrict__ w, uint64_t n, int sgn, int f, F *__restrict__ out,
    int aligned16) {
  constexpr int NT = B <= 31 ? 256 : 128, kPitch = kGroup + 1;
  constexpr int PER = 16 / sizeof(F);
  __shared__ F tile[NT * kPitch];
  const int tid = threadIdx.x;
  const uint64_t g = (uint64_t)blockIdx.x * NT + tid, e0 = (uint64_t)blockIdx.x * NT * kGroup;
  if (g * kGroup < n) {
    F *dst = tile + tid * kPitch;
    if constexpr (B <= 31) {
      uint32_t v[kGroup];
      codec::decode32<B>(w + g * B, sgn, v);
#pragma unroll
      for (int i = 0; i < kGroup; ++i) dst[i] = (F)ldexp((double)(int32_t)v[i], -f);
    } else {
      int64_t v[kGroup];
      codec::decode<B>(w + g * B, sgn, v);
#pragma unroll
      for (int i = 0; i < kGroup; ++i) dst[i] = (F)ldexp((double)v[i], -f);
    }
  }
  __syncthreads();
  if (aligned16 && e0 + (uint64_t)NT * kGroup <= n) {
#pragma unroll
    for (int j = 0; j < kGroup / PER; ++j) {
      const int q = (tid + j * NT) * PER;
      u32x4_t t;
      F *x = reinterpret_cast<F *>(&t);
#pragma unroll
      for (int u = 0; u < PER; ++u) x[u] = tile[q + u + (q >> 5)];
      __builtin_nontemporal_store(t, reinterpret_cast<u32x4_t *>(out + e0 + q));
    }
  } else {
    for (int q = tid; q < NT * kGroup; q += NT)
      if (e0 + q < n) out[e0 + q] = tile[q + (q >> 5)];
  }
}

template <typename F>
hipError_t launch_fx_range(const F *v, uint64_t n, int f, int bits, double qlo, double qhi,
                           uint32_t *out, uint64_t cap32, RangeSink sink, hipStream_t s) {
  const uint64_t ngroups = (cap32 + bits - 1) / bits;
  const int nt = bits <= 31 ? 256 : 128;
  const uint64_t grid = (ngroups + nt - 1) / nt;
  if (grid > 0x7fffffffull) return hipErrorInvalidValue;
  const int al = ((uintptr_t)v % 16) == 0;
  switch (bits) {
#define CCM_FX_RANGE(b)                                                                          \
  case b:                                                                                        \
    k_compress_fx_range<b, F>                                                                    \
        <<<(unsigned)grid, nt, 0, s>>>(v, n, f, qlo, qhi, out, cap32, sink, al);                 \
    break;
    CCM_WIDTH_CASES(CCM_FX_RANGE)
#undef CCM_FX_RANGE
    default: return hipErrorInvalidValue;
  }
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : launch_range_publish(sink, s);
}

template <typename F>
hipError_t launch_fx_decode(const uint32_t *w, uint64_t n, int bits, int sgn, int f, F *out,
                            hipStream_t s) {
  const uint64_t ngroups = (n + kGroup - 1) / kGroup;
  const int nt = bits <= 31 ? 256 : 128;
  const uint64_t grid = (ngroups + nt - 1) / nt;
  if (grid > 0x7fffffffull) return hipErrorInvalidValue;
  const int al = ((uintptr_t)out % 16) == 0;
  switch (bits) {
#define CCM_FX_DECODE(b)                                                            \
  case b:                                                                           \
    k_decompress_fx<b, F><<<(unsigned)grid, nt, 0, s>>>(w, n, sgn, f, out, al);     \
    break;
    CCM_WIDTH_CASES(CCM_FX_DECODE)
#undef CCM_FX_DECODE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

unsigned fx_grid(uint64_t n) {
  const uint64_t g = (n + 4ull * kFxThreads - 1) / (4ull * kFxThreads);
  return (unsigned)(g < 1 ? 1 : (g > 8192 ? 8192 : g));
}

}  // namespace

hipError_t launch_float_range(const void *v, int dtype, uint64_t n, RangeSink sink,
                              hipStream_t s) {
  const uint64_t per = 16ull * kFxThreads;  // four 16-byte loads of doubles a lane, a few times
  const uint64_t g = (n + per - 1) / per;
  const unsigned grid = (unsigned)(g < 1 ? 1 : (g > 4096 ? 4096 : g));
  const int al = ((uintptr_t)v % 16) == 0;
  if (dtype == CCM_F64)
    k_float_range<double><<<grid, kFxThreads, 0, s>>>((const double *)v, n, sink, al);
  else
    k_float_range<float><<<grid, kFxThreads, 0, s>>>((const float *)v, n, sink, al);
  return hipGetLastError();
}

hipError_t launch_float_sample(const void *v, int dtype, uint64_t n, RangeSink sink,
                               hipStream_t s) {
  if (dtype == CCM_F64)
    k_float_sample<double><<<kSampleBlocks, kFxThreads, 0, s>>>((const double *)v, n, sink);
  else
    k_float_sample<float><<<kSampleBlocks, kFxThreads, 0, s>>>((const float *)v, n, sink);
  return hipGetLastError();
}

hipError_t launch_compress_fx_range(const void *v, int dtype, uint64_t n, int frac_bits, int bits,
                                    double qlo, double qhi, uint32_t *out, uint64_t cap32,
                                    RangeSink sink, hipStream_t s) {
  if (dtype == CCM_F64)
    return launch_fx_range<double>((const double *)v, n, frac_bits, bits, qlo, qhi, out, cap32,
                                   sink, s);
  return launch_fx_range<float>((const float *)v, n, frac_bits, bits, qlo, qhi, out, cap32, sink,
                                s);
}

hipError_t launch_decompress_fx(const uint32_t *w, uint64_t n, int bits, int sgn, int frac_bits,
                                int dtype, void *out, hipStream_t s) {
  if (dtype == CCM_F64)
    return launch_fx_decode<double>(w, n, bits, sgn, frac_bits, (double *)out, s);
  return launch_fx_decode<float>(w, n, bits, sgn, frac_bits, (float *)out, s);
}

hipError_t launch_quantize(const void *v, int dtype, uint64_t n, int frac_bits, void *q,
                           int qdtype, RangeSink sink, hipStream_t s) {
  const unsigned g = fx_grid(n);
  if (dtype == CCM_F64 && qdtype == CCM_I64)
    k_quantize<double, int64_t><<<g, kFxThreads, 0, s>>>((const double *)v, n, frac_bits,
                                                         (int64_t *)q, sink);
  else if (dtype == CCM_F64)
    k_quantize<double, int32_t><<<g, kFxThreads, 0, s>>>((const double *)v, n, frac_bits,
                                                         (int32_t *)q, sink);
  else if (qdtype == CCM_I64)
    k_quantize<float, int64_t><<<g, kFxThreads, 0, s>>>((const float *)v, n, frac_bits,
                                                        (int64_t *)q, sink);
  else
    k_quantize<float, int32_t><<<g, kFxThreads, 0, s>>>((const float *)v, n, frac_bits,
                                                        (int32_t *)q, sink);
  return hipGetLastError();
}

hipError_t launch_compress_fx(const void *v, int dtype, uint64_t n, int frac_bits, int bits,
                              uint32_t *out, uint64_t cap32, hipStream_t s) {
  const uint64_t ngroups = (cap32 + bits - 1) / bits;
  const uint64_t grid = (ngroups + kFxTile - 1) / kFxTile;
  if (grid > 0x7fffffffull) return hipErrorInvalidValue;
  const int al = ((uintptr_t)v % 16) == 0;
  if (dtype == CCM_F64)
    k_compress_fx<double><<<(unsigned)grid, kFxTile, 0, s>>>((const double *)v, n, frac_bits,
                                                             bits, out, cap32, ngroups, al);
  else
    k_compress_fx<float><<<(unsigned)grid, kFxTile, 0, s>>>((const float *)v, n, frac_bits,
                                                            bits, out, cap32, ngroups, al);
  return hipGetLastError();
}

hipError_t launch_dequantize(const int64_t *q, uint64_t n, int frac_bits, int dtype, void *out,
                             hipStream_t s) {
  if (dtype == CCM_F64)
    k_dequantize<double><<<fx_grid(n), kFxThreads, 0, s>>>(q, n, frac_bits, (double *)out);
  else
    k_dequantize<float><<<fx_grid(n), kFxThreads, 0, s>>>(q, n, frac_bits, (float *)out);
  return hipGetLastError();
}

}  // namespace ccm
