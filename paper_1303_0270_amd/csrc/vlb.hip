// Method 2 of the paper (Variable Length Blocks): every element is stored in
// its own minimal width b_e, preceded by a fixed k-bit length field holding
// b_e, with k the bit-length of the largest b_e (Methods, "Method 2"; Eq. 16
// counts the bits).  Elements follow each other in row-major order, least
// significant bit first, straddling 64-bit bitstrings as in Method 1.
//
// The stream alone can only be read from its start.  For random access and
// data-parallel decoding the library keeps an index beside it:
//   row_bit[i]   (uint64, rows + 1 entries): stream bit where row i starts;
//                row_bit[rows] is the total bit count;
//   grp_off[i][g] (uint32, rows x ceil(cols/32)): bit offset of element
//                (i, 32g) from the start of row i.
// A "group" is 32 consecutive elements of one row (the last group of a row
// may be shorter).  A lane that owns a group knows where it starts and walks
// its 32 (length, value) pairs; where the next one starts depends on the
// length just read, so the walk is serial within a group and parallel across
// groups.
//
// Encoding reads the dense values twice.  The first pass gives the exact range
// (hence k and the sign rule) and, per group, the sum of the element widths
// under either sign rule; scans (within rows, then over rows) add k per
// element and turn the sums into the index.  In the packing pass a block
// assembles the bits of 128 consecutive groups in LDS (four elements a lane,
// eight lanes a group, placed with a prefix sum of their lengths) and writes
// them out: the words its stretch covers entirely with plain stores, the two
// it shares with its neighbours with atomic ORs into words zeroed before.
#include <hip/hip_runtime.h>

#include "ccm_internal.hpp"

namespace ccm {
namespace {

constexpr int kVG = 32;          // elements per index group
constexpr int kVThreads = 256;   // threads per block of every VLB kernel

__device__ __forceinline__ int bitlen64(uint64_t u) { return u ? 64 - __clzll((long long)u) : 0; }

// b_e of one value: Eq. 1 on the element when the matrix has no negative
// value; otherwise the smallest two's complement width holding it.
__device__ __forceinline__ int elem_width(int64_t v, int sgn) {
  if (!sgn) {
    const int L = bitlen64((uint64_t)v);
    return L > 1 ? L : 1;
  }
  const uint64_t m = v < 0 ? ~(uint64_t)v : (uint64_t)v;
  return 1 + bitlen64(m);
}

template <typename T>
__device__ __forceinline__ int64_t load_dense(const T *d, uint64_t e) {
  return (int64_t)d[e];
}

// nb (1..64) stream bits starting at bit p, zero-extended.  Reads words
// p/32 .. p/32 + 2, which stay inside the payload capacity for any field
// that starts inside the stream.
__device__ __forceinline__ uint64_t bits_at(const uint32_t *w, uint64_t p, int nb) {
  const uint64_t q = p >> 5;
  const int off = (int)(p & 31u);
  uint64_t v = ((uint64_t)w[q] | ((uint64_t)w[q + 1] << 32)) >> off;
  if (off + nb > 64) v |= (uint64_t)w[q + 2] << (64 - off);
  return v & mask64(nb);
}

// ---- four elements a lane -----------------------------------------------------
//
// Both passes over the dense values give lane t of a wave elements
// 32g + 4(t % 8) .. + 3 of group t / 8: two (int64) or one (int32) 16-byte
// loads that a wave's lanes lay side by side, a group's sums three shuffles
// apart instead of five, and the work of placing a pair shared by four.

constexpr int kQuad = 4;                      // elements per lane
constexpr int kLanes = kVG / kQuad;           // lanes per group
constexpr int kStepGroups = kVThreads / kLanes;  // groups a block takes per step

// Elements j0 .. j0 + 3 of row i, clamped into the row (what lies past its end
// is the caller's to drop): loads without branches, so that the compiler
// issues all of a lane's before it waits for the first.  VEC: rows and quads
// start on 16-byte boundaries and every quad lies wholly inside or outside.
template <bool VEC, typename T>
__device__ __forceinline__ void load_quad(const T *__restrict__ d, uint64_t i, int64_t j0,
                                          int64_t cols, T (&v)[kQuad]) {
  const T *p = d + i * (uint64_t)cols;
  if constexpr (VEC) {
    constexpr int N = kQuad * (int)sizeof(T) / 16;
    const uint4 *p4 = reinterpret_cast<const uint4 *>(p + (j0 < cols ? j0 : 0));
    uint4 r[N];
#pragma unroll
    for (int q = 0; q < N; ++q) r[q] = p4[q];
#pragma unroll
    for (int q = 0; q < kQuad; ++q) v[q] = reinterpret_cast<const T *>(r)[q];
  } else {
#pragma unroll
    for (int q = 0; q < kQuad; ++q) v[q] = p[j0 + q < cols ? j0 + q : cols - 1];
  }
}

template <typename T>
bool quads_aligned(const T *d, int64_t cols) {
  return (uintptr_t)d % 16 == 0 && cols % kQuad == 0;
}

// ---- pass 1: range, and element widths per group -------------------------------

// grp[group] = sum of the unsigned widths | sum of the two's complement widths
// << 16 (each at most 32 * 64).  The unsigned ones mean nothing in a matrix
// with a negative value, which takes the others.  Bound by memory; the range
// and the sums were a pass each before (206 + 280 us at 16384 x 8192 int64
// against 220 here, 4.9 TB/s).
template <bool VEC, typename T>
__global__ __launch_bounds__(kVThreads) void k_vlb_stats(const T *__restrict__ dense, int64_t rows,
                                                         int64_t cols, int64_t ngr,
                                                         uint32_t *__restrict__ grp,
                                                         RangeSink sink) {
  const uint64_t total = (uint64_t)rows * (uint64_t)ngr;
  const uint64_t step = (uint64_t)gridDim.x * kStepGroups;
  // group gi = (row i, group g of the row), advanced by the grid step with
  // one division up front
  const uint64_t di = step / (uint64_t)ngr, dg = step - di * (uint64_t)ngr;
  uint64_t gi = (uint64_t)blockIdx.x * kStepGroups + threadIdx.x / kLanes;
  uint64_t i = gi / (uint64_t)ngr, g = gi - i * (uint64_t)ngr;
  const int sub = threadIdx.x % kLanes;
  int64_t lo = INT64_MAX, hi = INT64_MIN;
  // kSteps grid steps per iteration, their loads issued before any is used
  constexpr int kSteps = 4;
  for (; gi < total; gi += kSteps * step) {
    T v[kSteps][kQuad];
    int live[kSteps];
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
      const bool valid = gi + u * step < total;
      const int64_t j0 = (int64_t)g * kVG + sub * kQuad;
      const int64_t left = valid ? cols - j0 : 0;
      live[u] = left >= kQuad ? kQuad : left > 0 ? (int)left : 0;
      load_quad<VEC>(dense, valid ? i : 0, j0, cols, v[u]);
      g += dg;
      i += di;
      if (g >= (uint64_t)ngr) {
        g -= (uint64_t)ngr;
        ++i;
      }
    }
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
      uint32_t sum = 0;
#pragma unroll
      for (int q = 0; q < kQuad; ++q) {
        if (q < live[u]) {
          const int64_t x = (int64_t)v[u][q];
          lo = x < lo ? x : lo;
          hi = x > hi ? x : hi;
          const uint32_t L = (uint32_t)bitlen64((uint64_t)(x ^ (x >> 63)));
          sum += (L > 1u ? L : 1u) + ((L + 1u) << 16);
        }
      }
#pragma unroll
      for (int m = kLanes / 2; m >= 1; m >>= 1) sum += (uint32_t)__shfl_xor((int)sum, m, kLanes);
      if (sub == 0 && gi + u * step < total) grp[gi + u * step] = sum;
    }
  }
  block_range_commit(lo, hi, 0, sink);
}

// ---- pass 2: scans ----------------------------------------------------------

// Inclusive block-wide scan of one value per thread (uint64), with the block
// total.  Every thread must call it.
template <int NT>
__device__ __forceinline__ uint64_t block_scan_incl(uint64_t v, uint64_t *total) {
  __shared__ uint64_t s_wave[NT / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint64_t o = __shfl_up(v, d, 64);
    if (lane >= d) v += o;
  }
  if (lane == 63) s_wave[wave] = v;
  __syncthreads();
  uint64_t before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) {
    const uint64_t s = s_wave[w];
    before += w < wave ? s : 0;
    all += s;
  }
  __syncthreads();  // s_wave is reused by the next call
  *total = all;
  return v + before;
}

// Row i's width sums (under the matrix's sign rule, k added per element) become
// exclusive offsets from the row start; the row's total goes to row_bit[i + 1]
// (the next kernel turns those into starts).  A wave per row, four groups a
// lane and step: no barrier between rows.  The longest group, which sizes the
// staging buffers of the other kernels, folds into the slots' maximum.
__global__ __launch_bounds__(kVThreads) void k_vlb_row_scan(int64_t rows, int64_t cols,
                                                            int64_t ngr, int k, int sgn,
                                                            uint32_t *__restrict__ grp,
                                                            uint64_t *__restrict__ row_bit,
                                                            RangeSink slots) {
  constexpr int kWaves = kVThreads / 64;
  const int lane = threadIdx.x & 63;
  uint32_t gmax = 0;
  for (int64_t i = (int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6); i < rows;
       i += (int64_t)gridDim.x * kWaves) {
    uint32_t *gp = grp + (uint64_t)i * (uint64_t)ngr;
    uint32_t carry = 0;  // a row holds fewer than 2^32 bits
    for (int64_t c0 = 0; c0 < ngr; c0 += 4 * 64) {
      const int64_t g0 = c0 + 4 * lane;
      uint32_t v[4], sum = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = gp[g0 + q < ngr ? g0 + q : ngr - 1];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t n = cols - (g0 + q) * kVG;  // elements from this group on
        v[q] = (sgn ? v[q] >> 16 : v[q] & 0xffffu) + (uint32_t)k * (uint32_t)(n < kVG ? n : kVG);
        v[q] = g0 + q < ngr ? v[q] : 0u;
        gmax = v[q] > gmax ? v[q] : gmax;
        sum += v[q];
      }
      uint32_t inc = sum;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = (uint32_t)__shfl_up((int)inc, d, 64);
        if (lane >= d) inc += o;
      }
      uint32_t at = carry + inc - sum;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (g0 + q < ngr) gp[g0 + q] = at;
        at += v[q];
      }
      carry += (uint32_t)__shfl((int)inc, 63, 64);
    }
    if (lane == 0) row_bit[i + 1] = carry;
  }
  block_range_commit(INT64_MAX, (int64_t)gmax, 0, slots);
}

// row_bit[0] = 0 and row_bit[i + 1] = sum of the first i + 1 row totals, by one
// block of 1024 threads that takes eight rows each at a time, read and written
// side by side through LDS; then the total and the longest group are published
// (vmin and vmax of the record).  16384 rows: 14 us (one row a thread and step
// 45, eight read straight from memory 20).
constexpr int kScanThreads = 1024, kScanPer = 8;
__global__ __launch_bounds__(kScanThreads) void k_vlb_rows_scan(int64_t rows,
                                                                uint64_t *__restrict__ row_bit,
                                                                RangeSink sink) {
  __shared__ uint64_t s_tot[kScanThreads * (kScanPer + 1)];
  const int t = threadIdx.x;
  uint64_t carry = 0;
  for (int64_t c0 = 0; c0 < rows; c0 += kScanThreads * kScanPer) {
    uint64_t v[kScanPer], sum = 0, tot = 0;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
      const int64_t i = c0 + q * kScanThreads + t;
      v[q] = i < rows ? row_bit[i + 1] : 0;
    }
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
      const int e = q * kScanThreads + t;
      s_tot[e + e / kScanPer] = v[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
      v[q] = s_tot[t * (kScanPer + 1) + q];
      sum += v[q];
    }
    uint64_t at = carry + block_scan_incl<kScanThreads>(sum, &tot) - sum;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
      at += v[q];
      s_tot[t * (kScanPer + 1) + q] = at;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) {
      const int e = q * kScanThreads + t;
      if (c0 + e < rows) row_bit[c0 + e + 1] = s_tot[e + e / kScanPer];
    }
    carry += tot;
    __syncthreads();
  }
  if (t == 0) {
    row_bit[0] = 0;
    atomicMin((long long *)&sink.slot->vmin, (long long)carry);
  }
  __threadfence_system();  // the row starts, before the record
  __syncthreads();
  if (t < 64) range_publish(sink);
}

// ---- pass 3: packing -----------------------------------------------------------

// Zeroes the words the packing blocks share (the first word of each stretch of
// kPackGroups groups) and everything from the last one to the capacity's end.
constexpr int kPackGroups = 128;

__global__ __launch_bounds__(kVThreads) void k_vlb_zero_shared(
    int64_t ngr, uint64_t total, const uint64_t *__restrict__ row_bit,
    const uint32_t *__restrict__ grp, uint64_t nbits, uint32_t *__restrict__ out, uint64_t cap32) {
  const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  const uint64_t stretches = (total + kPackGroups - 1) / kPackGroups;
  for (uint64_t b = t; b < stretches; b += stride) {
    const uint64_t gb = b * kPackGroups;
    out[(row_bit[gb / (uint64_t)ngr] + grp[gb]) >> 5] = 0;
  }
  for (uint64_t q = (nbits >> 5) + t; q < cap32; q += stride) out[q] = 0;
}

// Appends n (1..32) bits x (no bits past n set) to a bit string in LDS: whole
// words leave as they fill.  LDS atomics, since the first and last word of a
// lane's bits belong to its neighbours too.
struct BitAppender {
  uint32_t *word;
  uint64_t buf;
  int used;
  __device__ __forceinline__ void put(uint32_t x, int n) {
    buf |= (uint64_t)x << used;
    used += n;
    if (used >= 32) {
      atomicOr(word++, (uint32_t)buf);
      buf >>= 32;
      used -= 32;
    }
  }
};

// A block assembles the stream of kPackGroups consecutive groups (a
// contiguous stretch of bits [S, E)) in LDS, then writes it out.
//   * Each lane loads its four quads of elements (32 groups apart) and their
//     groups' start bits before placing any.  A quad's bits follow each other,
//     so a prefix sum over the eight lanes of a group places four pairs at
//     once, and the lane appends them through a 64-bit buffer: one LDS atomic
//     per word instead of up to three for each length and each value.
//   * Write-out: the words the stretch covers entirely are plain coalesced
//     stores; its first and last words, shared with the neighbouring blocks,
//     are atomic ORs into words zeroed before.
// Bound by vector instructions at short widths (about 25 an element).  16384 x
// 8192 int64, bit-lengths Beta(1, 32): 295 us; a lane per element, with
// the whole payload zeroed before (19 us), took 443.
template <bool VEC, typename T>
__global__ __launch_bounds__(kVThreads) void k_vlb_pack(const T *__restrict__ dense, int64_t rows,
                                                        int64_t cols, int64_t ngr, int k, int sgn,
                                                        const uint64_t *__restrict__ row_bit,
                                                        const uint32_t *__restrict__ grp,
                                                        uint64_t nbits,
                                                        uint32_t *__restrict__ out) {
  extern __shared__ uint32_t span[];
  const uint64_t total = (uint64_t)rows * (uint64_t)ngr;
  const int sub = threadIdx.x % kLanes;
  for (uint64_t gb = (uint64_t)blockIdx.x * kPackGroups; gb < total;
       gb += (uint64_t)gridDim.x * kPackGroups) {
    const uint64_t ge = gb + kPackGroups < total ? gb + kPackGroups : total;
    // (row, group) of this lane's first group; the others from it
    constexpr int kPackPer = kPackGroups / kStepGroups;
    const uint64_t gi0 = gb + threadIdx.x / kLanes;
    uint64_t i = gi0 / (uint64_t)ngr, g = gi0 - i * (uint64_t)ngr;
    T v[kPackPer][kQuad];
    uint64_t gstart[kPackPer];
    int live[kPackPer];
#pragma unroll
    for (int u = 0; u < kPackPer; ++u) {
      const uint64_t gi = gi0 + (uint64_t)u * kStepGroups;
      const int64_t j0 = (int64_t)g * kVG + sub * kQuad;
      const bool valid = gi < ge;
      const int64_t left = valid ? cols - j0 : 0;
      live[u] = left >= kQuad ? kQuad : left > 0 ? (int)left : 0;
      const uint64_t ic = valid ? i : 0;
      gstart[u] = row_bit[ic] + grp[valid ? gi : 0];
      load_quad<VEC>(dense, ic, j0, cols, v[u]);
      g += kStepGroups;
      while (g >= (uint64_t)ngr) {
        g -= (uint64_t)ngr;
        ++i;
      }
    }
    // stretch [S, E) of groups gb .. ge - 1
    const uint64_t S = row_bit[gb / (uint64_t)ngr] + grp[gb];
    const uint64_t E = ge < total ? row_bit[ge / (uint64_t)ngr] + grp[ge] : nbits;
    const uint64_t q0 = S >> 5;
    const int nwords = (int)(((E + 31u) >> 5) - q0);
    for (int w = threadIdx.x; w < nwords; w += blockDim.x) span[w] = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPackPer; ++u) {
      int b[kQuad];
      uint32_t len = 0;
#pragma unroll
      for (int q = 0; q < kQuad; ++q) {
        b[q] = q < live[u] ? elem_width((int64_t)v[u][q], sgn) : 0;
        len += q < live[u] ? (uint32_t)(k + b[q]) : 0u;
      }
      uint32_t inc = len;
#pragma unroll
      for (int d = 1; d < kLanes; d <<= 1) {
        const uint32_t o = (uint32_t)__shfl_up((int)inc, d, kLanes);
        if (sub >= d) inc += o;
      }
      if (live[u]) {
        const uint32_t pos = (uint32_t)(gstart[u] - q0 * 32u) + (inc - len);
        BitAppender bits{span + (pos >> 5), 0, (int)(pos & 31u)};
#pragma unroll
        for (int q = 0; q < kQuad; ++q) {
          if (q < live[u]) {
            const uint64_t m = (uint64_t)(int64_t)v[u][q] & mask64(b[q]);
            const uint32_t head = (uint32_t)b[q] | ((uint32_t)m << k);
            const int n = k + b[q];
            if (n <= 32) {
              bits.put(head, n);
            } else {
              bits.put(head, 32);
              const uint64_t rest = m >> (32 - k);
              if (n <= 64) {
                bits.put((uint32_t)rest, n - 32);
              } else {
                bits.put((uint32_t)rest, 32);
                bits.put((uint32_t)(rest >> 32), n - 64);
              }
            }
          }
        }
        if (bits.used && (uint32_t)bits.buf) atomicOr(bits.word, (uint32_t)bits.buf);
      }
    }
    __syncthreads();
    for (int w = threadIdx.x; w < nwords; w += blockDim.x) {
      const uint64_t q = q0 + (uint64_t)w;
      const uint32_t val = span[w];
      if (q * 32u >= S && q * 32u + 32u <= E)
        out[q] = val;
      else if (val)
        atomicOr(&out[q], val);
    }
    __syncthreads();  // the span is cleared for the next stretch
  }
}

// ---- decode, get ------------------------------------------------------------

// One (length, value) pair at stream bit *p; advances *p.
__device__ __forceinline__ int64_t vlb_read(const uint32_t *w, uint64_t *p, int k, int sgn) {
  const int b = (int)bits_at(w, *p, k);
  const uint64_t u = bits_at(w, *p + (uint64_t)k, b);
  *p += (uint64_t)(k + b);
  return sgn ? sext64(u, b) : (int64_t)u;
}

__global__ __launch_bounds__(kVThreads) void k_vlb_decode(const uint32_t *__restrict__ w,
                                                          const uint64_t *__restrict__ row_bit,
                                                          const uint32_t *__restrict__ grp,
                                                          int64_t rows, int64_t cols, int64_t ngr,
                                                          int k, int sgn, int64_t *__restrict__ out) {
  const uint64_t total = (uint64_t)rows * (uint64_t)ngr;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t gi = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; gi < total; gi += stride) {
    const int64_t i = (int64_t)(gi / (uint64_t)ngr);
    const int64_t g = (int64_t)(gi - (uint64_t)i * (uint64_t)ngr);
    uint64_t p = row_bit[i] + grp[gi];
    const int64_t j0 = g * kVG;
    const int n = cols - j0 < kVG ? (int)(cols - j0) : kVG;
    int64_t *dst = out + (uint64_t)i * (uint64_t)cols + (uint64_t)j0;
    for (int l = 0; l < n; ++l) dst[l] = vlb_read(w, &p, k, sgn);
  }
}

__global__ void k_vlb_get(const uint32_t *__restrict__ w, const uint64_t *__restrict__ row_bit,
                          const uint32_t *__restrict__ grp, int64_t ngr, int64_t i, int64_t j,
                          int k, int sgn, RangeHost *host, uint32_t seq) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const int64_t g = j / kVG;
  uint64_t p = row_bit[i] + grp[(uint64_t)i * (uint64_t)ngr + (uint64_t)g];
  int64_t v = 0;
  for (int64_t l = g * kVG; l <= j; ++l) v = vlb_read(w, &p, k, sgn);
  __hip_atomic_store(&host->vmin, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __hip_atomic_store(&host->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---- matvec ------------------------------------------------------------------

// General form: any k + b_e, int32 or int64 x.  Block (chunk c, row i) walks
// groups 256c .. 256c + 255 of row i, one per lane, reading the stream
// straight from memory; the block's sum goes to y[i] (atomically when a row
// has more than one chunk; y was zeroed).
template <typename XT>
__global__ __launch_bounds__(kVThreads) void k_vlb_mv_gen(
    const uint32_t *__restrict__ w, const uint64_t *__restrict__ row_bit,
    const uint32_t *__restrict__ grp, int64_t rows, int64_t cols, int64_t ngr, int k, int sgn,
    const XT *__restrict__ x, int64_t *__restrict__ y) {
  __shared__ uint64_t s_part[kVThreads / 64];
  const int64_t nchunk = (ngr + kVThreads - 1) / kVThreads;
  const uint64_t nblk = (uint64_t)rows * (uint64_t)nchunk;
  for (uint64_t bi = blockIdx.x; bi < nblk; bi += gridDim.x) {
    const int64_t i = (int64_t)(bi / (uint64_t)nchunk);
    const int64_t c = (int64_t)(bi - (uint64_t)i * (uint64_t)nchunk);
    const int64_t g = c * kVThreads + threadIdx.x;
    uint64_t acc = 0;
    if (g < ngr) {
      uint64_t p = row_bit[i] + grp[(uint64_t)i * (uint64_t)ngr + (uint64_t)g];
      const int64_t j0 = g * kVG;
      const int n = cols - j0 < kVG ? (int)(cols - j0) : kVG;
      for (int l = 0; l < n; ++l) {
        const int64_t a = vlb_read(w, &p, k, sgn);
        acc += (uint64_t)a * (uint64_t)(int64_t)x[j0 + l];
      }
    }
    const int64_t ws = wave_sum((int64_t)acc);
    if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = (uint64_t)ws;
    __syncthreads();
    if (threadIdx.x == 0) {
      uint64_t t = 0;
#pragma unroll
      for (int v = 0; v < kVThreads / 64; ++v) t += s_part[v];
      if (nchunk > 1)
        atomicAdd((unsigned long long *)&y[i], (unsigned long long)t);
      else
        y[i] = (int64_t)t;
    }
    __syncthreads();
  }
}

// Both of (a == b ? x0 : y0) and (a == b ? x1 : y1) from one compare and
// two v_cndmask.  As plain C the compiler turns the select of two values just
// read from LDS into a select of their addresses and demotes the chain state
// to scratch.
__device__ __forceinline__ void select_eq2(uint32_t a, uint32_t b, uint32_t x0, uint32_t y0,
                                           uint32_t x1, uint32_t y1, uint32_t &r0,
                                           uint32_t &r1) {
  asm("v_cmp_eq_u32 vcc, %2, %3\n\t"
      "v_cndmask_b32 %0, %5, %4, vcc\n\t"
      "v_cndmask_b32 %1, %7, %6, vcc"
      : "=&v"(r0), "=v"(r1)
      : "v"(a), "v"(b), "v"(x0), "v"(y0), "v"(x1), "v"(y1)
      : "vcc");
}

// 64 stream bits from bit pv of a staged stretch (reads three words).
__device__ __forceinline__ uint64_t lds_bits64(const uint32_t *seg, uint32_t pv) {
  const uint32_t q = pv >> 5;
  const uint32_t w0 = seg[q], w1 = seg[q + 1], w2 = seg[q + 2];
  const uint32_t lo = __builtin_amdgcn_alignbit(w1, w0, pv & 31u);
  const uint32_t hi = __builtin_amdgcn_alignbit(w2, w1, pv & 31u);
  return ((uint64_t)hi << 32) | lo;
}

// Staged form for int32 x on a 16-byte boundary, any widths.
//   * Block (panel p, row slice) owns groups [256 GPT p, 256 GPT (p + 1)) of
//     the rows it visits; lane t owns groups 256 GPT p + GPT t + u (u < GPT),
//     GPT independent chains (instruction-level parallelism in the serial
//     walks), and keeps their 32 GPT x values in registers for all rows.
//   * Per row the block copies the panel's stretch of the stream (contiguous:
//     the panel's groups follow each other) into LDS with 16-byte
//     memory-to-LDS loads (global_load_lds_dwordx4, no registers), issued
//     right after the walks of the previous row.  One buffer: a second one,
//     filled a row ahead, measured slower, since it halves the blocks per CU
//     and the other resident blocks already cover a block's copy.
//   * A chain keeps the two stream words around its position in registers
//     (w0 = word q, w1 = word q + 1).  Per element: a funnel shift
//     (v_alignbit) gives the 32 bits at the pair's start; the length is their
//     low k bits; the value is one bit-field extract of the same word
//     (sign-extending when signed) and the product one 32x32->64
//     multiply-add.  A pair of at most 32 bits moves the position by at most
//     one word, so the window advances with a select and ONE new LDS word per
//     element.  A longer pair (rare in the paper's bit-length distributions)
//     takes a branch that reads the 64 bits at the value's start, corrects
//     the product and reloads the window.
//   * Rows visited: blockIdx.y, blockIdx.y + gridDim.y, ... (resident
//     blocks only, so x is loaded once per block).  Wave partial sums of row
//     r are folded and stored after the barrier that opens row r + 1.
//   * CLAMP: some chain of the panel is shorter than 32 elements or absent
//     (ragged row end, partial panel); its walk then continues through bits
//     of the next group or past the stretch, with x = 0 for those elements,
//     and its reads are clamped inside the staged buffer.
template <bool SGN, int GPT, bool CLAMP, bool WIDE>
__global__ __launch_bounds__(kVThreads) void k_vlb_mv_lds(
    const uint32_t *__restrict__ w, const uint64_t *__restrict__ row_bit,
    const uint32_t *__restrict__ grp, int64_t rows, int64_t cols, int64_t ngr, int k,
    int seg_words, const int32_t *__restrict__ x, int64_t *__restrict__ y, int atomic_out) {
  extern __shared__ uint4 seg4[];
  // the stretch buffer (seg_words words), then the wave partial sums of two
  // rows
  uint64_t *s_part = (uint64_t *)((uint32_t *)seg4 + seg_words);
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t g0 = (int64_t)blockIdx.x * kVThreads * GPT;
  const int64_t ge = g0 + kVThreads * GPT < ngr ? g0 + kVThreads * GPT : ngr;
  const uint32_t kmask = (1u << k) - 1u;
  const uint32_t narrow = 32u - (uint32_t)k;  // largest b read from one 32-bit window
  const uint32_t qmax = (uint32_t)seg_words - 4u;
  const uint32_t pmax = qmax * 32u;
  const uint32_t pmaxw = ((uint32_t)seg_words - 5u) * 32u;  // four-word reads

  int32_t xr[GPT][kVG];
#pragma unroll
  for (int u = 0; u < GPT; ++u) {
    const int64_t c0 = (g0 + (int64_t)GPT * t + u) * kVG;
    if (c0 + kVG <= cols) {
      const int4 *xv = (const int4 *)(x + c0);
#pragma unroll
      for (int q = 0; q < kVG / 4; ++q) {
        const int4 v = xv[q];
        xr[u][4 * q] = v.x;
        xr[u][4 * q + 1] = v.y;
        xr[u][4 * q + 2] = v.z;
        xr[u][4 * q + 3] = v.w;
      }
    } else {
#pragma unroll
      for (int j = 0; j < kVG; ++j) xr[u][j] = c0 + j < cols ? x[c0 + j] : 0;
    }
  }

  // Row r's stage: its start bit, first staged word (16-byte aligned) and
  // 16-byte vector count; the lanes' raw group offsets (clamped loads,
  // branch-free) and the copy of the stretch into the buffer.
  uint64_t nb_base = 0, nb_ws = 0;
  uint32_t graw[GPT];
  auto stage = [&](int64_t r) {
    const uint64_t base = row_bit[r];
    const uint32_t *gr = grp + (uint64_t)r * (uint64_t)ngr;
    const uint64_t s = base + gr[g0];
    const uint64_t e = ge < ngr ? base + gr[ge] : row_bit[r + 1];
    const uint64_t ws = (s >> 5) & ~3ull;
    const uint64_t we = ((e + 31u) >> 5) + 2u;  // two guard words for the 64-bit reads
    const int nvec = (int)((we - ws + 3u) >> 2);
#pragma unroll
    for (int u = 0; u < GPT; ++u) {
      int64_t g = g0 + (int64_t)GPT * t + u;
      g = g < ngr ? g : ngr - 1;
      graw[u] = gr[g];
    }
    const uint4 *src = (const uint4 *)(w + ws);
    uint4 *dst = seg4;
    for (int v0 = 0; v0 < nvec; v0 += kVThreads) {
      const int v = v0 + t;
      if (v < nvec)
        __builtin_amdgcn_global_load_lds(
            (const void *)(src + v),
            (__attribute__((address_space(3))) void *)(dst + v0 + 64 * wave), 16, 0, 0);
    }
    nb_base = base;
    nb_ws = ws;
  };

  int64_t r = blockIdx.y;
  if (r < rows) stage(r);
  int cur = 0;
  int64_t prev = -1;  // row whose wave sums wait in s_part[cur ^ 1]
  while (r < rows) {
    __builtin_amdgcn_s_waitcnt(0);  // all counters to zero: this lane's copies have landed
    __syncthreads();                // everyone's copies have landed
    if (prev >= 0 && t == 0) {
      uint64_t sum = 0;
#pragma unroll
      for (int v = 0; v < kVThreads / 64; ++v) sum += s_part[4 * (cur ^ 1) + v];
      if (atomic_out)
        atomicAdd((unsigned long long *)&y[prev], (unsigned long long)sum);
      else
        y[prev] = (int64_t)sum;
    }
    uint32_t p[GPT];
#pragma unroll
    for (int u = 0; u < GPT; ++u) {
      const int64_t g = g0 + (int64_t)GPT * t + u;
      p[u] = g < ngr ? (uint32_t)(nb_base + graw[u] - nb_ws * 32u) : 0u;
    }
    const int64_t rn = r + gridDim.y;

    // x stays in 32-bit registers: without this the compiler hoists the
    // sign extensions out of the row loop and doubles the register count
#pragma unroll
    for (int u = 0; u < GPT; ++u)
#pragma unroll
      for (int j = 0; j < kVG; ++j) asm volatile("" : "+v"(xr[u][j]));

    const uint32_t *seg = (const uint32_t *)seg4;
    int64_t acc[GPT];
    // the window: words q, q + 1 around the position and q + 2 requested
    // ahead (a pair of at most 32 bits moves the position by at most a
    // word, so the next window is (w0, w1) or (w1, w2), never a word still
    // in flight)
    // The four-word walk keeps the four words at its (clamped) read
    // position q in w0..w3, and requests the next element's as soon as the
    // length is known, before the value and the product.
    uint32_t q[GPT], w0[GPT], w1[GPT], w2[GPT], w3[GPT];
#pragma unroll
    for (int u = 0; u < GPT; ++u) {
      acc[u] = 0;
      if constexpr (WIDE) {
        q[u] = CLAMP && p[u] > pmaxw ? pmaxw : p[u];
        const uint32_t qc = q[u] >> 5;
        w0[u] = seg[qc];
        w1[u] = seg[qc + 1];
        w2[u] = seg[qc + 2];
        w3[u] = seg[qc + 3];
      } else {
        q[u] = p[u] >> 5;
        w0[u] = seg[q[u]];
        w1[u] = seg[q[u] + 1];
        w2[u] = seg[q[u] + 2];
        w3[u] = 0u;
      }
    }
#pragma unroll
    for (int j = 0; j < kVG; ++j) {
#pragma unroll
      for (int u = 0; u < GPT; ++u) {
        if constexpr (WIDE) {
          // four words at the pair's start give 96 bits: the length and a
          // value of up to 64 bits, with no branch
          const uint32_t sh = q[u] & 31u;
          const uint32_t a0 = __builtin_amdgcn_alignbit(w1[u], w0[u], sh);
          const uint32_t a1 = __builtin_amdgcn_alignbit(w2[u], w1[u], sh);
          const uint32_t a2 = __builtin_amdgcn_alignbit(w3[u], w2[u], sh);
          const uint32_t b = a0 & kmask;
          p[u] += (uint32_t)k + b;
          // the next pair's words, requested before this one's value and
          // product (kept here: the scheduler would sink them to their use)
          q[u] = CLAMP && p[u] > pmaxw ? pmaxw : p[u];
          const uint32_t qc = q[u] >> 5;
          w0[u] = seg[qc];
          w1[u] = seg[qc + 1];
          w2[u] = seg[qc + 2];
          w3[u] = seg[qc + 3];
          __builtin_amdgcn_sched_barrier(0);
          const int nb = b < 64u ? (int)b : 64;
          const uint64_t lo = ((uint64_t)a1 << 32) | a0;
          uint64_t v = ((lo >> k) | ((uint64_t)a2 << (64 - k))) & mask64(nb);
          if (SGN) v = (uint64_t)sext64(v, nb > 0 ? nb : 1);
          acc[u] += (int64_t)(v * (uint64_t)(int64_t)xr[u][j]);
          asm volatile("" : "+v"(acc[u]));
          continue;
        }
        const uint32_t wv = __builtin_amdgcn_alignbit(w1[u], w0[u], p[u] & 31u);
        const uint32_t b = wv & kmask;
        int32_t a;
        if (SGN)
          a = opaque_i32(__builtin_amdgcn_sbfe((int32_t)wv, k, b));
        else
          a = (int32_t)__builtin_amdgcn_ubfe(wv, k, b);
        acc[u] += (int64_t)a * (int64_t)xr[u][j];
        // one v_add3 (the compiler otherwise keeps p + k apart for the rare
        // branch and spends two adds on every element)
        uint32_t pn;
        asm("v_add3_u32 %0, %1, %2, %3" : "=v"(pn) : "v"(p[u]), "s"((uint32_t)k), "v"(b));
        uint32_t qn = pn >> 5;
        if (CLAMP) qn = qn < qmax ? qn : qmax;
        // the word after the next window, requested as early as its address
        // is known (kept here: left to itself the scheduler sinks the
        // request to its use in the next element, which then waits for it)
        const uint32_t w2n = seg[qn + 2];
        __builtin_amdgcn_sched_barrier(0);
        uint32_t w0n, w1n;
        select_eq2(qn, q[u], w0[u], w1[u], w1[u], w2[u], w0n, w1n);
        if (__builtin_expect(b > narrow, 0)) {
          // the value runs past the 32 bits read: replace a by the full
          // value, and reload the window where the next pair starts
          uint32_t pv = p[u] + (uint32_t)k;
          if (CLAMP) pv = pv < pmax ? pv : pmax;
          const int nb = b < 64u ? (int)b : 64;
          uint64_t v = lds_bits64(seg, pv) & mask64(nb);
          if (SGN) v = (uint64_t)sext64(v, nb);
          int32_t xw = xr[u][j];
          asm volatile("" : "+v"(xw));  // sign-extend here, not hoisted
          acc[u] += (int64_t)((v - (uint64_t)(int64_t)a) * (uint64_t)(int64_t)xw);
          w0n = seg[qn];
          w1n = seg[qn + 1];
          // wait for these two here, on the rare path: a wait at the merge
          // would also wait for the prefetch on the common one
          __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
        }
        asm volatile("" : "+v"(acc[u]));  // accumulate in place, element by element
        w2[u] = w2n;
        w1[u] = w1n;
        w0[u] = w0n;
        q[u] = qn;
        p[u] = pn;
      }
    }
    int64_t tot = 0;
#pragma unroll
    for (int u = 0; u < GPT; ++u) tot += acc[u];
    tot = wave_sum(tot);
    if (lane == 0) s_part[4 * cur + wave] = (uint64_t)tot;
    __syncthreads();  // every walk is done before the copy overwrites the buffer
    if (rn < rows) stage(rn);
    prev = r;
    r = rn;
    cur ^= 1;
  }
  __syncthreads();
  if (prev >= 0 && t == 0) {
    uint64_t sum = 0;
#pragma unroll
    for (int v = 0; v < kVThreads / 64; ++v) sum += s_part[4 * (cur ^ 1) + v];
    if (atomic_out)
      atomicAdd((unsigned long long *)&y[prev], (unsigned long long)sum);
    else
      y[prev] = (int64_t)sum;
  }
}

int compute_units() {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0, n = 0;
    (void)hipGetDevice(&dev);
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        n < 1)
      n = 256;
    cus = n;
  }
  return cus;
}

constexpr size_t kMaxLds = 160 * 1024 - 64;

// A panel's stretch: at most 256 GPT gmax bits, plus the alignment of its
// first word down to 16 bytes, the two guard words after its last, the
// rounding to whole 16-byte vectors and the clamp margin.
int stage_words(uint64_t gmax, int gpt) {
  return (int)(((uint64_t)kVThreads * gpt * gmax + 31u) / 32u + 16u) & ~3;
}

// The stretch buffer and the wave partial sums of two rows.
size_t stage_lds(uint64_t gmax, int gpt) {
  return (size_t)stage_words(gmax, gpt) * 4u + 2u * (kVThreads / 64) * 8u;
}

template <bool SGN, int GPT, bool CLAMP, bool WIDE>
int resident_lds(size_t lds) {
  int occ = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_vlb_mv_lds<SGN, GPT, CLAMP, WIDE>,
                                                   kVThreads, lds) != hipSuccess ||
      occ < 1)
    occ = 1;
  return occ * compute_units();
}

template <bool SGN, int GPT, bool CLAMP, bool WIDE>
hipError_t launch_mv_lds(const VlbView &a, const int32_t *x, int64_t *y, hipStream_t s) {
  const int64_t per_panel = (int64_t)kVThreads * GPT;
  const int64_t npanels = (a.ngr + per_panel - 1) / per_panel;
  if (npanels > 65535) return hipErrorInvalidValue;
  const int seg_words = stage_words(a.gmax, GPT);
  const size_t lds = stage_lds(a.gmax, GPT);
  if (lds > kMaxLds) return hipErrorInvalidValue;
  static bool attr = false;
  if (!attr) {
    hipError_t e = hipFuncSetAttribute((const void *)k_vlb_mv_lds<SGN, GPT, CLAMP, WIDE>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds);
    if (e != hipSuccess) return e;
    attr = true;
  }
  if (npanels > 1) {
    hipError_t e = launch_fill_i64(y, (uint64_t)a.rows, 0, s);
    if (e != hipSuccess) return e;
  }
  int64_t gy = resident_lds<SGN, GPT, CLAMP, WIDE>(lds) / npanels;
  gy = gy < 1 ? 1 : (gy > a.rows ? a.rows : gy);
  if (gy > 65535) gy = 65535;
  dim3 grid((unsigned)npanels, (unsigned)gy);
  k_vlb_mv_lds<SGN, GPT, CLAMP, WIDE><<<grid, kVThreads, lds, s>>>(
      a.w, a.row_bit, a.grp, a.rows, a.cols, a.ngr, a.k, seg_words, x, y, npanels > 1 ? 1 : 0);
  return hipGetLastError();
}

template <bool SGN, int GPT, bool WIDE>
hipError_t launch_mv_lds_c(const VlbView &a, const int32_t *x, int64_t *y, hipStream_t s) {
  const bool clamp = (a.cols % ((int64_t)kVThreads * GPT * kVG)) != 0;
  return clamp ? launch_mv_lds<SGN, GPT, true, WIDE>(a, x, y, s)
               : launch_mv_lds<SGN, GPT, false, WIDE>(a, x, y, s);
}

// Staged matvec: one group per lane (256 groups of at most 32 * 71 bits
// always fit in LDS), or two when that keeps strictly more chains resident
// per CU (blocks per CU from registers and LDS, times 256 GPT).  At equal
// chain counts one group per lane measured faster: twice the waves to hide
// the LDS latency of the walks.  Matrices whose pairs average more than 24
// bits (so that most pairs pass 32 bits, as with uniform bit-lengths) take
// the branch-free four-word walk.
template <bool SGN, bool WIDE>
hipError_t launch_mv_staged_w(const VlbView &a, const int32_t *x, int64_t *y, hipStream_t s) {
  const int64_t chains1 = (int64_t)resident_lds<SGN, 1, true, WIDE>(stage_lds(a.gmax, 1));
  int64_t chains2 = 0;
  if (stage_lds(a.gmax, 2) <= kMaxLds)
    chains2 = 2 * (int64_t)resident_lds<SGN, 2, true, WIDE>(stage_lds(a.gmax, 2));
  return chains2 > chains1 ? launch_mv_lds_c<SGN, 2, WIDE>(a, x, y, s)
                           : launch_mv_lds_c<SGN, 1, WIDE>(a, x, y, s);
}

template <bool SGN>
hipError_t launch_mv_staged(const VlbView &a, const int32_t *x, int64_t *y, hipStream_t s) {
  const uint64_t n = (uint64_t)a.rows * (uint64_t)a.cols;
  return a.nbits > 24u * n ? launch_mv_staged_w<SGN, true>(a, x, y, s)
                           : launch_mv_staged_w<SGN, false>(a, x, y, s);
}

unsigned vgrid(uint64_t work, uint64_t per_block, unsigned cap) {
  uint64_t g = (work + per_block - 1) / per_block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (unsigned)g;
}

}  // namespace

uint64_t vlb_ngr(int64_t cols) { return ((uint64_t)cols + kVG - 1) / kVG; }

hipError_t launch_vlb_stats(const void *dense, int dtype, int64_t rows, int64_t cols,
                            uint32_t *grp, RangeSink sink, hipStream_t s) {
  const int64_t ngr = (int64_t)vlb_ngr(cols);
  const unsigned grid = vgrid((uint64_t)rows * (uint64_t)ngr, kStepGroups * 4, 4096);
  if (dtype == CCM_I64) {
    const int64_t *d = (const int64_t *)dense;
    if (quads_aligned(d, cols))
      k_vlb_stats<true><<<grid, kVThreads, 0, s>>>(d, rows, cols, ngr, grp, sink);
    else
      k_vlb_stats<false><<<grid, kVThreads, 0, s>>>(d, rows, cols, ngr, grp, sink);
  } else {
    const int32_t *d = (const int32_t *)dense;
    if (quads_aligned(d, cols))
      k_vlb_stats<true><<<grid, kVThreads, 0, s>>>(d, rows, cols, ngr, grp, sink);
    else
      k_vlb_stats<false><<<grid, kVThreads, 0, s>>>(d, rows, cols, ngr, grp, sink);
  }
  return hipGetLastError();
}

hipError_t launch_vlb_scan(int64_t rows, int64_t cols, int k, int sgn, uint32_t *grp,
                           uint64_t *row_bit, RangeSink sink, hipStream_t s) {
  const int64_t ngr = (int64_t)vlb_ngr(cols);
  const unsigned grid = vgrid((uint64_t)rows, kVThreads / 64, 2048);
  k_vlb_row_scan<<<grid, kVThreads, 0, s>>>(rows, cols, ngr, k, sgn, grp, row_bit,
                                            RangeSink{sink.slot, nullptr, nullptr, 0});
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_vlb_rows_scan<<<1, kScanThreads, 0, s>>>(rows, row_bit, sink);
  return hipGetLastError();
}

hipError_t launch_vlb_pack(const void *dense, int dtype, const VlbView &a, uint32_t *out,
                           uint64_t cap32, uint64_t nbits, hipStream_t s) {
  const uint64_t total = (uint64_t)a.rows * (uint64_t)a.ngr;
  k_vlb_zero_shared<<<vgrid((total + kPackGroups - 1) / kPackGroups, kVThreads, 1024), kVThreads,
                      0, s>>>(a.ngr, total, a.row_bit, a.grp, nbits, out, cap32);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // a stretch of kPackGroups groups spans at most kPackGroups * gmax bits
  // and one word more
  const int span_words = (int)(((uint64_t)kPackGroups * a.gmax + 31u) / 32u + 2u);
  const size_t lds = (size_t)span_words * 4u;
  if (lds > 64 * 1024) return hipErrorInvalidValue;
  const unsigned grid = vgrid(total, kPackGroups, 65536);
  if (dtype == CCM_I64) {
    const int64_t *d = (const int64_t *)dense;
    if (quads_aligned(d, a.cols))
      k_vlb_pack<true><<<grid, kVThreads, lds, s>>>(d, a.rows, a.cols, a.ngr, a.k, a.sgn,
                                                    a.row_bit, a.grp, nbits, out);
    else
      k_vlb_pack<false><<<grid, kVThreads, lds, s>>>(d, a.rows, a.cols, a.ngr, a.k, a.sgn,
                                                     a.row_bit, a.grp, nbits, out);
  } else {
    const int32_t *d = (const int32_t *)dense;
    if (quads_aligned(d, a.cols))
      k_vlb_pack<true><<<grid, kVThreads, lds, s>>>(d, a.rows, a.cols, a.ngr, a.k, a.sgn,
                                                    a.row_bit, a.grp, nbits, out);
    else
      k_vlb_pack<false><<<grid, kVThreads, lds, s>>>(d, a.rows, a.cols, a.ngr, a.k, a.sgn,
                                                     a.row_bit, a.grp, nbits, out);
  }
  return hipGetLastError();
}

hipError_t launch_vlb_decode(const VlbView &a, int64_t *out, hipStream_t s) {
  const unsigned grid = vgrid((uint64_t)a.rows * (uint64_t)a.ngr, kVThreads, 65536);
  k_vlb_decode<<<grid, kVThreads, 0, s>>>(a.w, a.row_bit, a.grp, a.rows, a.cols, a.ngr, a.k,
                                          a.sgn, out);
  return hipGetLastError();
}

hipError_t launch_vlb_get(const VlbView &a, int64_t i, int64_t j, RangeHost *host, uint32_t seq,
                          hipStream_t s) {
  k_vlb_get<<<1, 64, 0, s>>>(a.w, a.row_bit, a.grp, a.ngr, i, j, a.k, a.sgn, host, seq);
  return hipGetLastError();
}

hipError_t launch_vlb_matvec(const VlbView &a, const void *x, int xdtype, int64_t *y,
                             hipStream_t s) {
  const bool staged = xdtype == CCM_I32 && ((uintptr_t)x % 16) == 0;
  if (staged) {
    const int32_t *xi = (const int32_t *)x;
    return a.sgn ? launch_mv_staged<true>(a, xi, y, s) : launch_mv_staged<false>(a, xi, y, s);
  }
  const int64_t nchunk = (a.ngr + kVThreads - 1) / kVThreads;
  if (nchunk > 1) {
    hipError_t e = launch_fill_i64(y, (uint64_t)a.rows, 0, s);
    if (e != hipSuccess) return e;
  }
  const unsigned grid = vgrid((uint64_t)a.rows * (uint64_t)nchunk, 1, 65536);
  if (xdtype == CCM_I64)
    k_vlb_mv_gen<int64_t><<<grid, kVThreads, 0, s>>>(a.w, a.row_bit, a.grp, a.rows, a.cols, a.ngr,
                                                     a.k, a.sgn, (const int64_t *)x, y);
  else
    k_vlb_mv_gen<int32_t><<<grid, kVThreads, 0, s>>>(a.w, a.row_bit, a.grp, a.rows, a.cols, a.ngr,
                                                     a.k, a.sgn, (const int32_t *)x, y);
  return hipGetLastError();
}

}  // namespace ccm
