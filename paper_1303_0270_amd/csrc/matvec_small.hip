// y = A x for small SM-packed matrices: an element per lane, few instructions.
//
// A call on a small matrix is bound by latency: the launch, the trips to memory
// one after the other, and the fetch of the code itself, which for kernels that
// decode 32 fields at compile-time offsets is thousands of instructions that no
// earlier wave has brought in.  Here the width is a runtime value and the whole
// kernel a loop of a few dozen instructions:
//   * consecutive lanes take consecutive columns; a field is two words (three
//     above 32 bits) from its own address, x straight from memory, both with
//     eight elements' loads in flight;
//   * W waves share a row (a power of two, about eight elements a lane), their
//     sums meeting in LDS: no zero fill, no atomics, whatever the shape.
// 256 x 256, in us with a launch each: int64 x at b = 10 9.5 before and 3.5 now,
// which is what an empty kernel takes here; int32 x at b = 1, 4, 10 24.7, 7.9 and
// 6.7 before.
#include <hip/hip_runtime.h>

#include "ccm_internal.hpp"

namespace ccm {
namespace {

constexpr int kInFlight = 8;

// The field of `bits` bits at bit s of the words lo, mid (and hi above 32 bits),
// extended to 64.
template <bool WIDE>
__device__ __forceinline__ uint64_t small_field(uint32_t lo, uint32_t mid, uint32_t hi, uint32_t s,
                                                int bits, int sgn) {
  const uint32_t a = __builtin_amdgcn_alignbit(mid, lo, s);
  if constexpr (WIDE) {
    const uint64_t f = (a | (uint64_t)__builtin_amdgcn_alignbit(hi, mid, s) << 32) << (64 - bits);
    return sgn ? (uint64_t)((int64_t)f >> (64 - bits)) : f >> (64 - bits);
  } else {
    const uint32_t f = a << (32 - bits);
    return sgn ? (uint64_t)(int64_t)((int32_t)f >> (32 - bits)) : f >> (32 - bits);
  }
}

template <typename XT, bool WIDE, int UNR>
__global__ void k_matvec_small(const uint32_t *__restrict__ A, int64_t rows, int cols, int bits,
                               int sgn, int waves, const XT *__restrict__ x,
                               int64_t *__restrict__ y) {
  __shared__ uint64_t part[16];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int per_block = (int)(blockDim.x >> 6) / waves;  // rows
  const int64_t row = (int64_t)blockIdx.x * per_block + wave / waves;
  const int64_t r = row < rows ? row : rows - 1;
  const uint64_t bit0 = (uint64_t)r * (uint64_t)cols * (uint64_t)bits;
  const uint32_t *w = A + (bit0 >> 5);
  const uint32_t head = (uint32_t)(bit0 & 31u);
  const int step = 64 * waves;
  uint64_t acc = 0;
  for (int c0 = (wave & (waves - 1)) * 64 + lane; c0 - lane < cols; c0 += step * UNR) {
    uint32_t lo[UNR], mid[UNR], hi[UNR];
    XT xv[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int c = c0 + u * step < cols ? c0 + u * step : cols - 1;
      const uint64_t bit = head + (uint64_t)c * (uint32_t)bits;
      const uint32_t *p = w + (bit >> 5);
      lo[u] = p[0];
      mid[u] = p[1];
      if constexpr (WIDE) hi[u] = p[2];
      xv[u] = x[c];
    }
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int c = c0 + u * step;
      const uint32_t s = (head + (uint32_t)c * (uint32_t)bits) & 31u;
      const uint64_t a = small_field<WIDE>(lo[u], mid[u], hi[u], s, bits, sgn);
      const uint64_t prod = a * (uint64_t)(int64_t)xv[u];
      acc += c < cols ? prod : 0;
    }
  }
  uint64_t sum = (uint64_t)wave_sum((int64_t)acc);
  if (waves > 1) {
    if (lane == 0) part[wave] = sum;
    __syncthreads();
    if (wave & (waves - 1)) return;
    sum = 0;
    for (int v = 0; v < waves; ++v) sum += part[wave + v];
  }
  if (lane == 0 && row < rows) y[row] = (int64_t)sum;
}


// y = A^T x (or A x of a matrix unravelled by column) alike: a block owns 16
// columns and all rows, a wave four rows of them at a time; the 64 or fewer rows
// that a block has at once are eight steps apart in flight, and its sums meet in
// shuffles and LDS.
constexpr int kColsT = 16;

template <typename XT, bool WIDE>
__global__ __launch_bounds__(1024) void k_matvec_t_small(const uint32_t *__restrict__ A, int rows,
                                                         int64_t cols, int bits, int sgn,
                                                         const XT *__restrict__ x,
                                                         int64_t *__restrict__ y) {
  __shared__ uint64_t part[16][kColsT];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int waves = blockDim.x >> 6, step = 4 * waves;
  const int64_t col = (int64_t)blockIdx.x * kColsT + (lane & (kColsT - 1));
  const int64_t c = col < cols ? col : cols - 1;
  uint64_t acc = 0;
  for (int r0 = 4 * wave + lane / kColsT; r0 - lane / kColsT < rows; r0 += step * kInFlight) {
    uint32_t lo[kInFlight], mid[kInFlight], hi[kInFlight], s[kInFlight];
    XT xv[kInFlight];
#pragma unroll
    for (int u = 0; u < kInFlight; ++u) {
      const int r = r0 + u * step < rows ? r0 + u * step : rows - 1;
      const uint64_t bit = ((uint64_t)r * (uint64_t)cols + (uint64_t)c) * (uint32_t)bits;
      const uint32_t *p = A + (bit >> 5);
      s[u] = (uint32_t)bit & 31u;
      lo[u] = p[0];
      mid[u] = p[1];
      if constexpr (WIDE) hi[u] = p[2];
      xv[u] = x[r];
    }
#pragma unroll
    for (int u = 0; u < kInFlight; ++u) {
      const uint64_t a = small_field<WIDE>(lo[u], mid[u], hi[u], s[u], bits, sgn);
      const uint64_t prod = a * (uint64_t)(int64_t)xv[u];
      acc += r0 + u * step < rows ? prod : 0;
    }
  }
  acc += (uint64_t)__shfl_xor((long long)acc, 16, 64);
  acc += (uint64_t)__shfl_xor((long long)acc, 32, 64);
  if (lane < kColsT) part[wave][lane] = acc;
  __syncthreads();
  if (threadIdx.x < kColsT && col < cols) {
    uint64_t sum = 0;
    for (int v = 0; v < waves; ++v) sum += part[v][threadIdx.x];
    y[col] = (int64_t)sum;
  }
}

template <typename XT>
void launch_t(const uint32_t *w, int64_t rows, int64_t cols, int bits, int sgn, const XT *x,
              int64_t *y, hipStream_t s) {
  int waves = 1;
  while (waves < 16 && waves * 4 * kInFlight < rows) waves *= 2;
  const unsigned grid = (unsigned)((cols + kColsT - 1) / kColsT);
  auto k = bits > 32 ? k_matvec_t_small<XT, true> : k_matvec_t_small<XT, false>;
  k<<<grid, 64 * waves, 0, s>>>(w, (int)rows, cols, bits, sgn, x, y);
}

template <typename XT, bool WIDE>
void launch(const uint32_t *w, int64_t rows, int cols, int bits, int sgn, const XT *x, int64_t *y,
            hipStream_t s) {
  int waves = 1;
  while (waves < 16 && waves * 64 * kInFlight < cols) waves *= 2;
  const int threads = waves > 4 ? waves * 64 : 256;
  const int per_block = threads / 64 / waves;
  const unsigned grid = (unsigned)((rows + per_block - 1) / per_block);
  // narrow matrices: no more loads than a row has elements for
  auto k = cols <= 64    ? k_matvec_small<XT, WIDE, 1>
           : cols <= 128 ? k_matvec_small<XT, WIDE, 2>
           : cols <= 256 ? k_matvec_small<XT, WIDE, 4>
                         : k_matvec_small<XT, WIDE, kInFlight>;
  k<<<grid, threads, 0, s>>>(w, rows, cols, bits, sgn, waves, x, y);
}

}  // namespace

hipError_t launch_matvec_small(const uint32_t *w, int64_t rows, int64_t cols, int bits, int sgn,
                               const void *x, int xdtype, int64_t *y, hipStream_t s) {
  if (xdtype == CCM_I32) {
    const int32_t *xi = (const int32_t *)x;
    if (bits > 32)
      launch<int32_t, true>(w, rows, (int)cols, bits, sgn, xi, y, s);
    else
      launch<int32_t, false>(w, rows, (int)cols, bits, sgn, xi, y, s);
  } else {
    const int64_t *xl = (const int64_t *)x;
    if (bits > 32)
      launch<int64_t, true>(w, rows, (int)cols, bits, sgn, xl, y, s);
    else
      launch<int64_t, false>(w, rows, (int)cols, bits, sgn, xl, y, s);
  }
  return hipGetLastError();
}

hipError_t launch_matvec_t_small(const uint32_t *w, int64_t rows, int64_t cols, int bits, int sgn,
                                 const void *x, int xdtype, int64_t *y, hipStream_t s) {
  if (xdtype == CCM_I32)
    launch_t<int32_t>(w, rows, cols, bits, sgn, (const int32_t *)x, y, s);
  else
    launch_t<int64_t>(w, rows, cols, bits, sgn, (const int64_t *)x, y, s);
  return hipGetLastError();
}

}  // namespace ccm
