// Instantiations of the limb GEMM for one limb count of A (each gemm_l*.hip
// compiles one).
#pragma once

#include <limits>
#include <type_traits>

#include "gemm_limb.hpp"

namespace ccm {
namespace limb {

// Tiles of eight waves, about 256 x 256 stacked outputs: 128 to 144
// accumulator registers a wave, 112 to 160 KB of LDS (one block per CU).
template <int LA, int LB, typename OT, bool CORR>
hipError_t launch_one(const GemmArgs &p, hipStream_t s) {
  if constexpr (LA == 3 && LB == 3)
    return launch_tile<LA, LB, 3, 3, 2, 4, OT, CORR>(p, s);
  else if constexpr (LA == 3)
    return launch_tile<LA, LB, 3, 2, 2, 4, OT, CORR>(p, s);
  else if constexpr (LB >= 3)
    return launch_tile<LA, LB, 2, LB, 4, 2, OT, CORR>(p, s);
  else
    return launch_tile<LA, LB, 4, 2, 2, 4, OT, CORR>(p, s);
}

template <int LA>
hipError_t launch_pass_la(const GemmArgs &p, int lb, int out32, hipStream_t s) {
  if constexpr (LA == 1) {
    if (lb == 1) {
      if (!p.radd && !p.cadd && out32) return launch_one<1, 1, int32_t, false>(p, s);
      return out32 ? launch_one<1, 1, int32_t, true>(p, s) : launch_one<1, 1, int64_t, true>(p, s);
    }
  }
  // Six limbs or more are never asked for an int32 C (matmul_fast_bytes).
#define CCM_LB(n)                                                                \
  if (lb == n) {                                                                 \
    if constexpr (LA + n < 6) {                                                  \
      if (out32) return launch_one<LA, n, int32_t, true>(p, s);                  \
    }                                                                            \
    return out32 ? hipErrorInvalidValue : launch_one<LA, n, int64_t, true>(p, s); \
  }
  if constexpr (LA > 1) {
    CCM_LB(1)
  }
  CCM_LB(2)
  if constexpr (LA <= 3) {
    CCM_LB(3)
  }
  if constexpr (LA <= 2) {
    CCM_LB(4)
  }
#undef CCM_LB
  return hipErrorInvalidValue;
}

}  // namespace limb
}  // namespace ccm
