// The product with up to 64 columns for A of 25 to 31 bits (see gemm_narrow.hpp).
#include "gemm_narrow.hpp"

namespace ccm {
namespace limb {

hipError_t launch_narrow_4(const SkinnyArgs &p, int abits, int waves, hipStream_t s) {
  switch (abits) {
    case 25: return launch_narrow_b<25>(p, waves, s);
    case 26: return launch_narrow_b<26>(p, waves, s);
    case 27: return launch_narrow_b<27>(p, waves, s);
    case 28: return launch_narrow_b<28>(p, waves, s);
    case 29: return launch_narrow_b<29>(p, waves, s);
    case 30: return launch_narrow_b<30>(p, waves, s);
    case 31: return launch_narrow_b<31>(p, waves, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace limb
}  // namespace ccm
