// matvec dispatch over the field width (instantiations live in matvec_w*.hip).
#include "ccm_internal.hpp"

namespace ccm {
namespace mv {
hipError_t launch_widths_1(const uint32_t *, int64_t, int64_t, int, int, const void *, int,
                           int64_t *, hipStream_t);
hipError_t launch_widths_2(const uint32_t *, int64_t, int64_t, int, int, const void *, int,
                           int64_t *, hipStream_t);
hipError_t launch_widths_3(const uint32_t *, int64_t, int64_t, int, int, const void *, int,
                           int64_t *, hipStream_t);
hipError_t launch_widths_4(const uint32_t *, int64_t, int64_t, int, int, const void *, int,
                           int64_t *, hipStream_t);
}  // namespace mv

hipError_t launch_matvec_small(const uint32_t *, int64_t, int64_t, int, int, const void *, int,
                               int64_t *, hipStream_t);

// Where an element per lane is the faster way (matvec_small.hip).  Measured
// against the kernels below, in us at b = 4, 10, 16, 24, 40 (int32 x over 31
// bits unless noted):
//   * up to 128 columns, as many rows as a launch of a wave a row holds (2^26):
//     8192 x 128 8.9 9.0 4.5 5.0 6.7 against 3.6; 300000 x 128 210 239 77 78 168
//     against 62 to 65; past 128 columns 20 to 50% is lost at b >= 16 (100000 x
//     300 30, 31 against 47).
//   * up to 2^20 elements: 256 x 256 7.9 6.7 3.5 3.8 4.4 against 3.5, int64 x
//     8.8 9.5 6.3 4.7 5.1 against 3.5; 1000 x 1003 5.1 6.1 3.9 4.5 4.9 against
//     3.5.  Below b = 16 up to 1.5 * 2^20 (1200 x 1200 5.0 5.9 against 4.7, but
//     b = 16 4.4 against 4.9), where 1448 x 1448 is even.
//   * few wide rows of wide fields, which leave most CUs without a row: int32 x
//     at b > 16, up to 512 rows and 2^22 elements: 128 x 16384 at b = 24, 31, 40
//     20 31 23 against 6.2, 300 x 10000 13 21 17 against 9 to 11.
static bool small_matvec(int64_t rows, int64_t cols, int bits, int xdtype) {
  if (cols <= 128) return launch_fits(((uint64_t)rows + 3) / 4, 256);  // four rows a block
  const uint64_t n = (uint64_t)rows * (uint64_t)cols;  // below 2^63 in a valid descriptor
  if (cols <= 16384 && n <= (bits < 16 ? 3ull << 19 : 1ull << 20)) return true;
  return xdtype == CCM_I32 && bits > 16 && rows <= 512 && cols <= 32768 && n <= 1ull << 22;
}

hipError_t launch_matvec(const uint32_t *w, int64_t rows, int64_t cols, int bits, int sgn,
                         const void *x, int xdtype, int64_t *y, hipStream_t s) {
  if (small_matvec(rows, cols, bits, xdtype))
    return launch_matvec_small(w, rows, cols, bits, sgn, x, xdtype, y, s);
  if (bits <= 16) return mv::launch_widths_1(w, rows, cols, bits, sgn, x, xdtype, y, s);
  if (bits <= 32) return mv::launch_widths_2(w, rows, cols, bits, sgn, x, xdtype, y, s);
  if (bits <= 48) return mv::launch_widths_3(w, rows, cols, bits, sgn, x, xdtype, y, s);
  return mv::launch_widths_4(w, rows, cols, bits, sgn, x, xdtype, y, s);
}

}  // namespace ccm
