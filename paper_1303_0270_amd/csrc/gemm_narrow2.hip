// The product with up to 64 columns for A of 9 to 16 bits (see gemm_narrow.hpp).
#include "gemm_narrow.hpp"

namespace ccm {
namespace limb {

hipError_t launch_narrow_2(const SkinnyArgs &p, int abits, int waves, hipStream_t s) {
  switch (abits) {
    case 9: return launch_narrow_b<9>(p, waves, s);
    case 10: return launch_narrow_b<10>(p, waves, s);
    case 11: return launch_narrow_b<11>(p, waves, s);
    case 12: return launch_narrow_b<12>(p, waves, s);
    case 13: return launch_narrow_b<13>(p, waves, s);
    case 14: return launch_narrow_b<14>(p, waves, s);
    case 15: return launch_narrow_b<15>(p, waves, s);
    case 16: return launch_narrow_b<16>(p, waves, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace limb
}  // namespace ccm
