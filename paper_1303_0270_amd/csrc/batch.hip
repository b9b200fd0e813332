// Batched matvec: y_t = A_t x_t for many SM-packed matrices of uneven shapes
// and widths in one persistent kernel launch (optionally a captured HIP graph;
// matrices of a few long rows of wide fields in a second one, k_batch_few).
//
// Host planner (ccm_batch_create): every matrix is cut into items of
// `tile_rows` rows (a per-width tuning table, JSON written by the autotuner, or
// built-in defaults; more rows for narrow matrices of a large batch, fewer for
// wide ones of a small batch), the items
// sorted by size class, largest first, and by width within a class: the sizes
// shrink towards the end, where the blocks have to finish together, and a block
// still keeps running one width's code for most of its time.  (By width first,
// the last items were the largest: 4096 matrices of 32..2048 squared, b = 1..24,
// took 1452 us where this order takes 1416.)
//
// Kernel: persistent blocks.  For an item, the block stages the digits of the
// matrix's x in LDS, then each wave takes tiles of 16 rows through the matrix
// cores (mv_tile.hpp).  Widths above 32, and payloads off a 16-byte boundary,
// use a runtime-width decoder.
//
// Bound by memory, and in narrow widths by what an item costs besides (its
// descriptors, x and the barriers).  2048 matrices of 32..2048 squared, in us,
// with a lane per group of a row and sums by shuffles, and now:
//   b = 1: 540, 140    b = 4: 595, 273    b = 8: 673, 466
//   b = 12: 864, 670   b = 16: 1049, 842  b = 24: 1274, 1209 (5.5 TB/s)
// and the 4096 of mixed widths 1610, 1366 (5.05 TB/s).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <sstream>
#include <string>
#include <vector>

#include "ccm.h"
#include "ccm_internal.hpp"
#include "matvec_impl.hpp"
#include "mv_tile.hpp"

namespace ccm {
namespace bt {

constexpr int kThreads = 256;
constexpr int kMaxCols = 8192;  // widest matrix a batch accepts (x is staged whole in LDS)

struct Mat {
  const uint32_t *w;
  const void *x;
  int64_t *y;
  int64_t rows, cols;
  int32_t bits, sgn;
};

struct Item {
  int32_t mat;
  int32_t row0;
  int32_t nrows;
  int32_t pad;
};

// x as it is, eight loads in flight per lane.
__device__ __forceinline__ void stage_words(const int32_t *__restrict__ x, int cols, int32_t *xs) {
  for (int c0 = threadIdx.x; c0 < cols; c0 += kThreads * 8) {
    int32_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = x[c0 + u * kThreads < cols ? c0 + u * kThreads : cols - 1];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (c0 + u * kThreads < cols) xs[c0 + u * kThreads] = v[u];
  }
}

// Rows of fields wider than 32 bits, at a runtime width: an element per lane, x
// from LDS, two elements in flight (64 columns apart, or of two rows where a row has
// no more than that).  Bound by the loads' latency.  us, x from memory and one
// element at a time, and so, at 40 bits: 8 of 100000 x 16 252 and 142, 8 of 100000 x
// 128 523 and 349, 4000 of 4 x 4000 424 and 162.
__device__ void item_rows_rt(const Mat &m, int row0, int nrows, const int32_t *x) {
  constexpr int kWaves = kThreads / 64;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int cols = (int)m.cols, left = 64 - m.bits;
  const mt::global_ptr<uint32_t> w = mt::as_global(m.w);
  const int dr = cols <= 64 ? kWaves : 0, dc = cols <= 64 ? 0 : 64;
  for (int rr = wave; rr < nrows; rr += kWaves + dr) {
    uint64_t acc[2] = {0, 0};
    for (int c0 = lane; c0 - lane < cols; c0 += 64 + dc) {
      uint32_t lo[2], mid[2], hi[2], s[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int c = c0 + u * dc < cols ? c0 + u * dc : cols - 1;
        const int r = rr + u * dr < nrows ? rr + u * dr : nrows - 1;
        const uint64_t bit =
            ((uint64_t)(row0 + r) * (uint64_t)cols + (uint64_t)c) * (uint64_t)m.bits;
        s[u] = (uint32_t)bit & 31u;
        lo[u] = w[bit >> 5];
        mid[u] = w[(bit >> 5) + 1];
        hi[u] = w[(bit >> 5) + 2];
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (c0 + u * dc < cols) {
          const uint64_t f = ((uint64_t)__builtin_amdgcn_alignbit(mid[u], lo[u], s[u]) |
                              (uint64_t)__builtin_amdgcn_alignbit(hi[u], mid[u], s[u]) << 32)
                             << left;
          const uint64_t a = m.sgn ? (uint64_t)((int64_t)f >> left) : f >> left;
          acc[u] += a * (uint64_t)(int64_t)x[c0 + u * dc];
        }
      }
    }
    if (!dr) acc[0] += acc[1];
    const int64_t tot = wave_sum((int64_t)acc[0]);
    if (lane == 0) m.y[(int64_t)row0 + rr] = tot;
    if (rr + dr >= nrows || !dr) continue;
    const int64_t next = wave_sum((int64_t)acc[1]);
    if (lane == 0) m.y[(int64_t)row0 + rr + dr] = next;
  }
}

// 2^this waves share a tile in an item of so many rows: one tile or two leave no
// wave without work (16 x 8000 at 24 bits: 26 us, 54 by one wave).
__device__ __forceinline__ int share_of(int nrows) {
  static_assert(kThreads == 256, "four waves");
  return nrows <= mt::kTileRows ? 2 : nrows <= 2 * mt::kTileRows ? 1 : 0;
}

// parts: 16 sums per wave, for an item whose tiles are shared.
__device__ __forceinline__ void dispatch(const Mat &m, const Item &it, const uint8_t *xd,
                                         uint64_t xsum, uint8_t *bufs, uint64_t *parts) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t ntile = ((int64_t)it.nrows + mt::kTileRows - 1) / mt::kTileRows;
  const uint32_t flip = mt::top_flip(m.bits, m.sgn);
  const uint64_t add = mt::tile_alpha(m.bits, m.sgn) * xsum;
  const uint64_t cap = 4u * cap_words32((uint64_t)m.rows * (uint64_t)m.cols, m.bits);
  switch (m.bits) {
#define CCM_B(b)                                                                               \
  case b:                                                                                      \
    mt::tiles<b>(m.w, cap, (int)m.cols, it.row0, (int64_t)it.row0 + it.nrows, wave,            \
                 kThreads / 64, ntile, flip, xd, add, bufs + wave * mt::Unit<b>::bytes, m.y,   \
                 share_of(it.nrows), parts + wave * mt::kTileRows);                            \
    return;
    CCM_WIDTH_CASES_32(CCM_B)
#undef CCM_B
    default:
      return;
  }
}

__global__ void k_counter_reset(int *counter, int first) { *counter = first; }

// A block takes items blockIdx + r gridDim for the first `rounds` rounds, then
// the next one by the counter: atomics on one address return one per 12 ns
// whatever the items hold (35,000 items of 128 rows at b = 1: 440 us of them),
// and by the second half of a sorted list there is still enough left to level
// the blocks.  The mix of widths: all by the counter 1378 us, half 1366, three
// quarters 1403, none 1438.
//
// The exit test is block-uniform (item indices from the counter are handed over
// through LDS).  A block stops at its first index past the end, so every block
// exits.
__global__ __launch_bounds__(kThreads) void k_batch(const Mat *__restrict__ mats,
                                                    const Item *__restrict__ items, int nitems,
                                                    int *counter, int rounds, int buf_bytes) {
  // the waves' buffers, then the digit rows of the widest matrix's x
  extern __shared__ __align__(16) uint8_t lds[];
  uint8_t *xd = lds + buf_bytes;
  __shared__ int s_item[2];
  __shared__ uint64_t s_sum[kThreads / 64], s_part[kThreads / 64 * mt::kTileRows];
  // The next item's index is requested when an item starts and read when it
  // ends, so the atomic's round trip overlaps the item's work.
  int next = 0;
  int it = blockIdx.x;
  for (int round = 1; it < nitems; ++round) {
    if (round >= rounds && threadIdx.x == 0) next = atomicAdd(counter, 1);
    const Item item = items[it];
    const Mat m = mats[item.mat];
    if (m.bits <= 32 && (uintptr_t)m.w % 16 == 0) {
      const uint64_t part = mt::stage_x<kThreads>((const int32_t *)m.x, (int)m.cols,
                                                  mt::spread_of(m.bits), xd);
      const uint64_t ws = (uint64_t)wave_sum((int64_t)part);
      if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = ws;
      __syncthreads();
      uint64_t xsum = 0;
#pragma unroll
      for (int v = 0; v < kThreads / 64; ++v) xsum += s_sum[v];
      dispatch(m, item, xd, xsum, lds, s_part);
      if (const int share = share_of(item.nrows)) {
        __syncthreads();
        if ((int)threadIdx.x < item.nrows) {
          const int tile = threadIdx.x / mt::kTileRows, row = threadIdx.x % mt::kTileRows;
          uint64_t sum = mt::tile_alpha(m.bits, m.sgn) * xsum;
          for (int v = 0; v < 1 << share; ++v)
            sum += s_part[((tile << share) + v) * mt::kTileRows + row];
          m.y[(int64_t)item.row0 + threadIdx.x] = (int64_t)sum;
        }
      }
    } else {
      int32_t *xs = reinterpret_cast<int32_t *>(xd);  // five digit rows hold more
      stage_words((const int32_t *)m.x, (int)m.cols, xs);
      __syncthreads();
      item_rows_rt(m, item.row0, item.nrows, xs);
    }
    if (round < rounds) {
      it += gridDim.x;
      __syncthreads();  // xd is rewritten by the next item
    } else {
      // the other slot: slower waves may still be reading the last one
      if (threadIdx.x == 0) s_item[round & 1] = next;
      __syncthreads();
      it = __builtin_amdgcn_readfirstlane(s_item[round & 1]);
    }
  }
}

// Few long rows of wide fields: a tile of 16 rows decodes as much for one of them as
// for sixteen.  A block takes a matrix, a wave a row at a time, a lane a group of 32
// fields; x in LDS with a lane's 32 values on 36 words.  us, 4000 of 1 x 4000 and 4 x
// 4000, in tiles and so: 24 bits 164 and 28, 168 and 44; 32 bits 217 and 30, 236 and
// 63.  At 16 bits and below the tiles are no slower.
constexpr int kFewRows = 8, kFewCols = 1024, kPitch = kGroup + 4;

template <int B, bool SGN>
__device__ __forceinline__ void few_rows(const Mat &m, const int32_t *xs) {
  const int lane = threadIdx.x & 63, ng = (int)((m.cols + kGroup - 1) / kGroup);
  const mt::global_ptr<uint32_t> w = mt::as_global(m.w);
  for (int r = threadIdx.x >> 6; r < (int)m.rows; r += kThreads / 64) {
    const uint64_t bit = (uint64_t)r * (uint64_t)m.cols * B;
    const int sh = (int)(bit & 31u);
    uint64_t acc = 0;
    for (int j = lane; j < ng; j += 64) {
      uint32_t ww[B + 1];
#pragma unroll
      for (int k = 0; k <= B; ++k) ww[k] = w[(bit >> 5) + (uint64_t)j * B + k];
#pragma unroll
      for (int k = 0; k < B; ++k) ww[k] = __builtin_amdgcn_alignbit(ww[k + 1], ww[k], sh);
      acc += mv::group_dot_wide<B, SGN, int32_t>(ww, xs + j * kPitch);
    }
    const int64_t sum = wave_sum((int64_t)acc);
    if (lane == 0) m.y[r] = sum;
  }
}

__global__ __launch_bounds__(kThreads) void k_batch_few(const Mat *__restrict__ mats,
                                                        const Item *__restrict__ items) {
  __shared__ __align__(16) int32_t xs[kMaxCols / kGroup * kPitch];
  const Mat m = mats[items[blockIdx.x].mat];
  const int cols = (int)m.cols, padded = (cols + kGroup - 1) / kGroup * kGroup;
  const mt::global_ptr<int32_t> x = mt::as_global((const int32_t *)m.x);
  for (int c0 = threadIdx.x; c0 < padded; c0 += kThreads * 8) {
    int32_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = x[c0 + u * kThreads < cols ? c0 + u * kThreads : cols - 1];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int c = c0 + u * kThreads;
      if (c < padded) xs[(c >> 5) * kPitch + (c & 31)] = c < cols ? v[u] : 0;
    }
  }
  __syncthreads();
  switch (2 * m.bits + (m.sgn ? 1 : 0)) {
#define CCM_FEW(b)                                          \
  case 2 * b: few_rows<b, false>(m, xs); return;            \
  case 2 * b + 1: few_rows<b, true>(m, xs); return;
    CCM_FEW(17) CCM_FEW(18) CCM_FEW(19) CCM_FEW(20) CCM_FEW(21) CCM_FEW(22) CCM_FEW(23)
    CCM_FEW(24) CCM_FEW(25) CCM_FEW(26) CCM_FEW(27) CCM_FEW(28) CCM_FEW(29) CCM_FEW(30)
    CCM_FEW(31) CCM_FEW(32)
#undef CCM_FEW
    default: return;
  }
}

inline bool takes_few(const Mat &m) {
  return m.rows <= kFewRows && m.cols >= kFewCols && m.bits > 16 && m.bits <= 32;
}

}  // namespace bt
}  // namespace ccm

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

using ccm::bt::Item;
using ccm::bt::Mat;

// Launch shape of a batch whose widest matrix has `cols` columns and whose fields
// have the `widths` (bit b: b bits) among those up to 32: LDS for the digit rows of
// x and the waves' buffers, and as many blocks as are resident with it.
namespace {
struct Shape {
  int lds = 0, bufs = 0, grid = 0;
  // rounds of items that the blocks take by their own index
  int rounds(size_t items) const { return 1 + (int)(items / grid) / 2; }
};
}  // namespace

struct ccm_batch {
  int n = 0;
  int32_t xdtype = CCM_I32;
  std::vector<Mat> mats;  // host copy (x, y filled by set_io)
  std::vector<Item> items;
  uint64_t packed_bytes = 0;
  int32_t max_bits = 0;
  Mat *d_mats = nullptr;
  Item *d_items = nullptr;
  int *d_counter = nullptr;
  int few = 0;  // matrices that k_batch_few takes
  Shape shape;
  hipStream_t cap_stream = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  bool io_set = false;
};

namespace {

struct TuneEntry {
  int tile_rows = 256;
};

// Defaults: small widths need more rows per item to amortize staging x.
TuneEntry default_tune(int bits) {
  TuneEntry t;
  t.tile_rows = bits <= 4 ? 512 : bits <= 12 ? 256 : 128;
  return t;
}

// Reads {"widths": {"<b>": {"tile_rows": r}, ...}}, other fields ignored; any
// parse problem leaves the defaults in place.
void load_tune(const char *path, TuneEntry table[65]) {
  for (int b = 1; b <= 64; ++b) table[b] = default_tune(b);
  if (!path) return;
  std::ifstream f(path);
  if (!f) return;
  std::stringstream ss;
  ss << f.rdbuf();
  const std::string s = ss.str();
  for (int b = 1; b <= 64; ++b) {
    const std::string key = "\"" + std::to_string(b) + "\"";
    size_t p = s.find(key);
    if (p == std::string::npos) continue;
    const size_t end = s.find('}', p);
    auto field = [&](const char *name, int *out) {
      const size_t q = s.find(name, p);
      if (q == std::string::npos || q > end) return;
      const size_t c = s.find(':', q);
      if (c == std::string::npos || c > end) return;
      const int v = std::atoi(s.c_str() + c + 1);
      if (v > 0) *out = v;
    };
    field("\"tile_rows\"", &table[b].tile_rows);
    if (table[b].tile_rows < 1) table[b].tile_rows = 1;
  }
}

int hip_status(hipError_t e) {
  if (e == hipSuccess) return CCM_OK;
  if (std::getenv("CCM_LOG")) std::fprintf(stderr, "ccm batch: %s\n", hipGetErrorString(e));
  return e == hipErrorOutOfMemory ? CCM_E_NOMEM : CCM_E_DEVICE;
}

int check_batch_descs(const ccm_desc *as, int32_t n) {
  for (int t = 0; t < n; ++t) {
    const ccm_desc &d = as[t];
    int32_t b = 0, s = 0;
    if (!d.payload || d.rows < 1 || d.cols < 1 || ccm_width(d.vmin, d.vmax, &b, &s) != CCM_OK ||
        b != d.bits || s != d.is_signed || d.words != ccm_words(d.rows, d.cols, d.bits))
      return CCM_E_INVAL;
    if (d.cols > ccm::bt::kMaxCols || d.rows > 0x7fffffff) return CCM_E_UNSUPPORTED;
  }
  return CCM_OK;
}

// Work list: items of tile_rows rows.  Where that gives every one of `blocks`
// blocks four or more, an item of fewer than 64 KB takes up to four times the
// rows: below that, what an item costs besides its payload shows (2048 matrices
// of 32..2048 squared, items of 128 and 512 rows: b = 1 211 and 140 us, b = 8
// 482 and 466, but b = 24 1209 and 1225; 64 matrices, which fill the blocks
// barely once, 36 and 38 us at b = 4, 47 and 80 at b = 16).  Fields past 32 bits
// are decoded one by one, next to which an item costs little: theirs stay within
// 128 rows.  Where the list leaves blocks idle, items of more than kHalveCols
// columns of wide fields, whose tiles a wave walks for long, are halved up to four
// times (128 rows: to 16, which the waves of a block then share), as long as that
// gives no block more than one item and the list has `room`: 1 of 300 x 8192 at 24
// bits 94 and 26 us, 20 of 300 x 8000 96 and 42.
struct Plan {
  int64_t count;  // items of tile_rows rows: what a workspace has to hold
  int few;        // matrices for k_batch_few, one item each at the end of the list
};
constexpr int64_t kHalveCols = 3000;

Plan plan_items(const std::vector<Mat> &mats, const TuneEntry *table, int blocks, int64_t room,
                std::vector<Item> *items) {
  items->clear();
  auto rows_of = [&](const Mat &d, int halved) {
    const int64_t rows = table[d.bits].tile_rows, tile = ccm::mt::kTileRows;
    const bool fixed = halved == 0 || rows <= tile || d.cols <= kHalveCols || d.bits <= 16;
    return fixed ? rows : std::max(rows >> halved, tile);
  };
  auto count_of = [&](int halved) {
    int64_t n = 0;
    for (const Mat &d : mats) n += (d.rows - 1) / rows_of(d, halved) + 1;
    return n;
  };
  Plan plan{count_of(0), 0};
  const int most = plan.count >= 4 * (int64_t)blocks ? 4 : 1;
  int halved = 0;
  while (halved < 4 && count_of(halved + 1) <= std::min<int64_t>(blocks, room)) ++halved;
  for (size_t t = 0; t < mats.size(); ++t) {
    const Mat &d = mats[t];
    if (ccm::bt::takes_few(d)) continue;
    int64_t rows = rows_of(d, halved);
    const int64_t limit = rows * most;
    while (rows < limit && (uint64_t)rows * d.cols * d.bits < (64u << 10) * 8u &&
           (d.bits <= 32 || rows <= 64))
      rows *= 2;
    for (int64_t r = 0; r < d.rows; r += rows) {
      const int nr = (int)std::min<int64_t>(rows, d.rows - r);
      items->push_back(Item{(int32_t)t, (int32_t)r, nr, 0});
    }
  }
  auto bits_of = [&](const Item &x) {
    return (uint64_t)x.nrows * (uint64_t)mats[x.mat].cols * (uint64_t)mats[x.mat].bits;
  };
  std::stable_sort(items->begin(), items->end(), [&](const Item &x, const Item &y) {
    const Mat &a = mats[x.mat], &c = mats[y.mat];
    const uint64_t sa = bits_of(x), sc = bits_of(y);
    const int la = __builtin_clzll(sa), lc = __builtin_clzll(sc);  // size classes: powers of two
    if (la != lc) return la < lc;
    if (a.bits != c.bits) return a.bits < c.bits;
    return sa > sc;
  });
  for (size_t t = 0; t < mats.size(); ++t)
    if (ccm::bt::takes_few(mats[t])) {
      items->push_back(Item{(int32_t)t, 0, (int32_t)mats[t].rows, 0});
      ++plan.few;
    }
  return plan;
}

// The kernels of a planned list whose tables are on the device.
hipError_t launch_items(const Shape &shape, const Mat *mats, const Item *items, int64_t n, int few,
                        int *counter, hipStream_t s) {
  const int64_t tiled = n - few;
  if (tiled) {
    const int rounds = shape.rounds((size_t)tiled);
    ccm::bt::k_counter_reset<<<1, 1, 0, s>>>(counter, rounds * shape.grid);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    ccm::bt::k_batch<<<shape.grid, ccm::bt::kThreads, shape.lds, s>>>(
        mats, items, (int)tiled, counter, rounds, shape.bufs);
  }
  if (few) ccm::bt::k_batch_few<<<few, ccm::bt::kThreads, 0, s>>>(mats, items + tiled);
  return hipGetLastError();
}

constexpr int kShapes = 4;
Shape launch_shape(int64_t cols, uint64_t widths) {
  Shape p;
  for (int b = 1; b <= 32; ++b)
    if (widths >> b & 1u)
      p.bufs = std::max(p.bufs, (ccm::bt::kThreads / 64) * ccm::mt::unit_bytes(b));
  p.lds = p.bufs + ccm::mt::x_lds((int)cols);
  (void)hipFuncSetAttribute(reinterpret_cast<const void *>(ccm::bt::k_batch),
                            hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
  int occ = 0, dev = 0, cus = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, ccm::bt::k_batch, ccm::bt::kThreads,
                                                   (size_t)p.lds) != hipSuccess ||
      occ < 1)
    occ = 1;
  (void)hipGetDevice(&dev);
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus < 1)
    cus = 256;
  p.grid = occ * cus;
  return p;
}

}  // namespace

// Reusable device workspace for batches whose matrices change on every launch
// (the serving loop): a ring of slots, each with pinned host staging, device
// tables and a completion event that guards its reuse.
struct ccm_batch_ws {
  struct Slot {
    Mat *h_mats = nullptr, *d_mats = nullptr;
    Item *h_items = nullptr, *d_items = nullptr;
    int *d_counter = nullptr;
    hipEvent_t done = nullptr;
    bool used = false;
  };
  int max_mats = 0;
  int64_t max_items = 0;
  Shape shapes[kShapes];  // by the widest matrix: up to 1024, 2048, 4096, 8192 columns
  int next = 0;
  TuneEntry table[65];
  std::vector<Slot> slots;
  std::vector<Mat> mats;
  std::vector<Item> items;
};

namespace {
void free_ws(ccm_batch_ws *w) {
  for (auto &s : w->slots) {
    if (s.h_mats) (void)hipHostFree(s.h_mats);
    if (s.h_items) (void)hipHostFree(s.h_items);
    if (s.d_mats) (void)hipFree(s.d_mats);
    if (s.d_items) (void)hipFree(s.d_items);
    if (s.d_counter) (void)hipFree(s.d_counter);
    if (s.done) (void)hipEventDestroy(s.done);
  }
  delete w;
}
}  // namespace

extern "C" {

int ccm_batch_create(const ccm_desc *as, int32_t n, int32_t xdtype, const char *tune_json,
                     ccm_batch **out) {
  if (!as || n < 1 || !out) return CCM_E_INVAL;
  if (xdtype != CCM_I32) return CCM_E_UNSUPPORTED;
  int rc = check_batch_descs(as, n);
  if (rc != CCM_OK) return rc;
  TuneEntry table[65];
  load_tune(tune_json, table);
  ccm_batch *b = new ccm_batch();
  b->n = n;
  b->xdtype = xdtype;
  b->mats.resize(n);
  for (int t = 0; t < n; ++t) {
    const ccm_desc &d = as[t];
    b->mats[t] = Mat{(const uint32_t *)d.payload, nullptr, nullptr, d.rows, d.cols, d.bits,
                     d.is_signed};
    b->packed_bytes += 8u * d.words;
    b->max_bits = std::max(b->max_bits, d.bits);
  }
  int64_t max_cols = 1;
  for (const Mat &m : b->mats) max_cols = std::max(max_cols, m.cols);
  uint64_t widths = 0;
  for (const Mat &m : b->mats) widths |= m.bits <= 32 ? 1ull << m.bits : 0u;
  b->shape = launch_shape(max_cols, widths);
  b->few = plan_items(b->mats, table, b->shape.grid, INT64_MAX, &b->items).few;
  rc = hip_status(hipMalloc(&b->d_mats, sizeof(Mat) * n));
  if (rc == CCM_OK) rc = hip_status(hipMalloc(&b->d_items, sizeof(Item) * b->items.size()));
  if (rc == CCM_OK) rc = hip_status(hipMalloc(&b->d_counter, 256));
  if (rc == CCM_OK)
    rc = hip_status(hipMemcpy(b->d_items, b->items.data(), sizeof(Item) * b->items.size(),
                              hipMemcpyHostToDevice));
  if (rc == CCM_OK) rc = hip_status(hipMemcpy(b->d_mats, b->mats.data(), sizeof(Mat) * n,
                                              hipMemcpyHostToDevice));
  if (rc == CCM_OK) rc = hip_status(hipStreamCreateWithFlags(&b->cap_stream, hipStreamNonBlocking));
  if (rc != CCM_OK) {
    ccm_batch_destroy(b);
    return rc;
  }
  *out = b;
  return CCM_OK;
}

int ccm_batch_set_io(ccm_batch *b, const void *const *xs, int64_t *const *ys, void *stream) {
  if (!b || !xs || !ys) return CCM_E_INVAL;
  for (int t = 0; t < b->n; ++t) {
    if (!xs[t] || !ys[t]) return CCM_E_INVAL;
    b->mats[t].x = xs[t];
    b->mats[t].y = ys[t];
  }
  // from pageable memory: the runtime stages the bytes before returning, and
  // the copy is ordered before later work on `stream`
  int rc = hip_status(hipMemcpyAsync(b->d_mats, b->mats.data(), sizeof(Mat) * b->n,
                                     hipMemcpyHostToDevice, (hipStream_t)stream));
  if (rc == CCM_OK) b->io_set = true;
  return rc;
}

static int batch_enqueue(ccm_batch *b, hipStream_t s) {
  return hip_status(launch_items(b->shape, b->d_mats, b->d_items, (int64_t)b->items.size(), b->few,
                                 b->d_counter, s));
}

int ccm_batch_matvec(ccm_batch *b, int32_t use_graph, void *stream) {
  if (!b) return CCM_E_INVAL;
  if (!b->io_set) return CCM_E_INVAL;
  hipStream_t s = (hipStream_t)stream;
  if (!use_graph) return batch_enqueue(b, s);
  if (!b->exec) {
    int rc = hip_status(hipStreamBeginCapture(b->cap_stream, hipStreamCaptureModeThreadLocal));
    if (rc != CCM_OK) return rc;
    rc = batch_enqueue(b, b->cap_stream);
    hipGraph_t g = nullptr;
    const int rc2 = hip_status(hipStreamEndCapture(b->cap_stream, &g));
    if (rc != CCM_OK || rc2 != CCM_OK) {
      if (g) (void)hipGraphDestroy(g);
      return rc != CCM_OK ? rc : rc2;
    }
    b->graph = g;
    rc = hip_status(hipGraphInstantiate(&b->exec, g, nullptr, nullptr, 0));
    if (rc != CCM_OK) return rc;
  }
  return hip_status(hipGraphLaunch(b->exec, s));
}

int ccm_batch_info(const ccm_batch *b, int64_t *items, uint64_t *packed_bytes,
                   int32_t *max_bits) {
  if (!b) return CCM_E_INVAL;
  if (items) *items = (int64_t)b->items.size();
  if (packed_bytes) *packed_bytes = b->packed_bytes;
  if (max_bits) *max_bits = b->max_bits;
  return CCM_OK;
}

int ccm_batch_ws_create(int32_t max_mats, int64_t max_items, int32_t slots, const char *tune_json,
                        ccm_batch_ws **out) {
  if (max_mats < 1 || max_items < 1 || slots < 1 || slots > 64 || !out) return CCM_E_INVAL;
  ccm_batch_ws *w = new ccm_batch_ws();
  w->max_mats = max_mats;
  w->max_items = max_items;
  load_tune(tune_json, w->table);
  w->slots.resize(slots);
  int rc = CCM_OK;
  for (auto &sl : w->slots) {
    if (rc == CCM_OK) rc = hip_status(hipHostMalloc((void **)&sl.h_mats, sizeof(Mat) * max_mats,
                                                    hipHostMallocDefault));
    if (rc == CCM_OK) rc = hip_status(hipHostMalloc((void **)&sl.h_items,
                                                    sizeof(Item) * max_items,
                                                    hipHostMallocDefault));
    if (rc == CCM_OK) rc = hip_status(hipMalloc((void **)&sl.d_mats, sizeof(Mat) * max_mats));
    if (rc == CCM_OK) rc = hip_status(hipMalloc((void **)&sl.d_items, sizeof(Item) * max_items));
    if (rc == CCM_OK) rc = hip_status(hipMalloc((void **)&sl.d_counter, 256));
    if (rc == CCM_OK) rc = hip_status(hipEventCreateWithFlags(&sl.done, hipEventDisableTiming));
  }
  for (int i = 0; rc == CCM_OK && i < kShapes; ++i)
    w->shapes[i] = launch_shape(ccm::bt::kMaxCols >> (kShapes - 1 - i), ~0ull);
  if (rc != CCM_OK) {
    free_ws(w);
    return rc;
  }
  *out = w;
  return CCM_OK;
}

int ccm_batch_ws_destroy(ccm_batch_ws *w) {
  if (!w) return CCM_E_INVAL;
  for (auto &sl : w->slots)
    if (sl.used) (void)hipEventSynchronize(sl.done);
  free_ws(w);
  return CCM_OK;
}

int ccm_batch_matvec_dyn(ccm_batch_ws *w, const ccm_desc *as, const void *const *xs,
                         int64_t *const *ys, int32_t n, void *stream) {
  if (!w || !as || !xs || !ys || n < 1) return CCM_E_INVAL;
  if (n > w->max_mats) return CCM_E_NOMEM;
  int rc = check_batch_descs(as, n);
  if (rc != CCM_OK) return rc;
  w->mats.resize(n);
  for (int t = 0; t < n; ++t) {
    if (!xs[t] || !ys[t]) return CCM_E_INVAL;
    const ccm_desc &d = as[t];
    w->mats[t] = Mat{(const uint32_t *)d.payload, xs[t], ys[t], d.rows, d.cols, d.bits,
                     d.is_signed};
  }
  int64_t max_cols = 1;
  for (const Mat &m : w->mats) max_cols = std::max(max_cols, m.cols);
  int i = 0;
  while (max_cols > (ccm::bt::kMaxCols >> (kShapes - 1 - i))) ++i;
  const Shape &shape = w->shapes[i];
  const Plan plan = plan_items(w->mats, w->table, shape.grid, w->max_items, &w->items);
  if (plan.count > w->max_items) return CCM_E_NOMEM;
  ccm_batch_ws::Slot &sl = w->slots[w->next];
  w->next = (w->next + 1) % (int)w->slots.size();
  if (sl.used) {
    rc = hip_status(hipEventSynchronize(sl.done));  // its previous upload has been consumed
    if (rc != CCM_OK) return rc;
  }
  std::memcpy(sl.h_mats, w->mats.data(), sizeof(Mat) * n);
  std::memcpy(sl.h_items, w->items.data(), sizeof(Item) * w->items.size());
  hipStream_t s = (hipStream_t)stream;
  rc = hip_status(hipMemcpyAsync(sl.d_mats, sl.h_mats, sizeof(Mat) * n, hipMemcpyHostToDevice, s));
  if (rc == CCM_OK)
    rc = hip_status(hipMemcpyAsync(sl.d_items, sl.h_items, sizeof(Item) * w->items.size(),
                                   hipMemcpyHostToDevice, s));
  if (rc != CCM_OK) return rc;
  rc = hip_status(launch_items(shape, sl.d_mats, sl.d_items, (int64_t)w->items.size(), plan.few,
                               sl.d_counter, s));
  if (rc != CCM_OK) return rc;
  rc = hip_status(hipEventRecord(sl.done, s));
  sl.used = (rc == CCM_OK);
  return rc;
}

int ccm_batch_destroy(ccm_batch *b) {
  if (!b) return CCM_E_INVAL;
  if (b->exec) (void)hipGraphExecDestroy(b->exec);
  if (b->graph) (void)hipGraphDestroy(b->graph);
  if (b->cap_stream) (void)hipStreamDestroy(b->cap_stream);
  if (b->d_mats) (void)hipFree(b->d_mats);
  if (b->d_items) (void)hipFree(b->d_items);
  if (b->d_counter) (void)hipFree(b->d_counter);
  delete b;
  return CCM_OK;
}

}  // extern "C"
