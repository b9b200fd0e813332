// The narrow-B product for A of 25 to 31 bits (see gemm_skinny.hpp).
#include "gemm_skinny.hpp"

namespace ccm {
namespace limb {

hipError_t launch_skinny_4(const SkinnyArgs &p, int abits, int nb, hipStream_t s) {
  switch (abits) {
    case 25: return launch_skinny_b<25>(p, nb, s);
    case 26: return launch_skinny_b<26>(p, nb, s);
    case 27: return launch_skinny_b<27>(p, nb, s);
    case 28: return launch_skinny_b<28>(p, nb, s);
    case 29: return launch_skinny_b<29>(p, nb, s);
    case 30: return launch_skinny_b<30>(p, nb, s);
    case 31: return launch_skinny_b<31>(p, nb, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace limb
}  // namespace ccm
