// The narrow-B product for A of 1 to 8 bits (see gemm_skinny.hpp).
#include "gemm_skinny.hpp"

namespace ccm {
namespace limb {

hipError_t launch_skinny_1(const SkinnyArgs &p, int abits, int nb, hipStream_t s) {
  switch (abits) {
    case 1: return launch_skinny_b<1>(p, nb, s);
    case 2: return launch_skinny_b<2>(p, nb, s);
    case 3: return launch_skinny_b<3>(p, nb, s);
    case 4: return launch_skinny_b<4>(p, nb, s);
    case 5: return launch_skinny_b<5>(p, nb, s);
    case 6: return launch_skinny_b<6>(p, nb, s);
    case 7: return launch_skinny_b<7>(p, nb, s);
    case 8: return launch_skinny_b<8>(p, nb, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace limb
}  // namespace ccm
