// The product with up to 64 columns for A of 17 to 24 bits (see gemm_narrow.hpp).
#include "gemm_narrow.hpp"

namespace ccm {
namespace limb {

hipError_t launch_narrow_3(const SkinnyArgs &p, int abits, int waves, hipStream_t s) {
  switch (abits) {
    case 17: return launch_narrow_b<17>(p, waves, s);
    case 18: return launch_narrow_b<18>(p, waves, s);
    case 19: return launch_narrow_b<19>(p, waves, s);
    case 20: return launch_narrow_b<20>(p, waves, s);
    case 21: return launch_narrow_b<21>(p, waves, s);
    case 22: return launch_narrow_b<22>(p, waves, s);
    case 23: return launch_narrow_b<23>(p, waves, s);
    case 24: return launch_narrow_b<24>(p, waves, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace limb
}  // namespace ccm
