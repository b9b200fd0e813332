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
      uint64_t a = __builtin_amdgcn_alignbit(mid[u], lo[u], s);
      if constexpr (WIDE) {
        a |= (uint64_t)__builtin_amdgcn_alignbit(hi[u], mid[u], s) << 32;
        a = sgn ? (uint64_t)((int64_t)(a << (64 - bits)) >> (64 - bits))
                : a << (64 - bits) >> (64 - bits);
      } else {
        const uint32_t f = (uint32_t)a << (32 - bits);
        a = sgn ? (uint64_t)(int64_t)((int32_t)f >> (32 - bits)) : f >> (32 - bits);
      }
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

}  // namespace ccm
