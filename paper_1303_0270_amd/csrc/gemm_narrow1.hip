// The product with up to 64 columns for A of 1 to 8 bits (see gemm_narrow.hpp).
#include "gemm_narrow.hpp"

namespace ccm {
namespace limb {

hipError_t launch_narrow_1(const SkinnyArgs &p, int abits, int waves, hipStream_t s) {
  switch (abits) {
    case 1: return launch_narrow_b<1>(p, waves, s);
    case 2: return launch_narrow_b<2>(p, waves, s);
    case 3: return launch_narrow_b<3>(p, waves, s);
    case 4: return launch_narrow_b<4>(p, waves, s);
    case 5: return launch_narrow_b<5>(p, waves, s);
    case 6: return launch_narrow_b<6>(p, waves, s);
    case 7: return launch_narrow_b<7>(p, waves, s);
    case 8: return launch_narrow_b<8>(p, waves, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace limb
}  // namespace ccm
