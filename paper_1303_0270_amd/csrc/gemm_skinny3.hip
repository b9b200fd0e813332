// The narrow-B product for A of 17 to 24 bits (see gemm_skinny.hpp).
#include "gemm_skinny.hpp"

namespace ccm {
namespace limb {

hipError_t launch_skinny_3(const SkinnyArgs &p, int abits, int nb, hipStream_t s) {
  switch (abits) {
    case 17: return launch_skinny_b<17>(p, nb, s);
    case 18: return launch_skinny_b<18>(p, nb, s);
    case 19: return launch_skinny_b<19>(p, nb, s);
    case 20: return launch_skinny_b<20>(p, nb, s);
    case 21: return launch_skinny_b<21>(p, nb, s);
    case 22: return launch_skinny_b<22>(p, nb, s);
    case 23: return launch_skinny_b<23>(p, nb, s);
    case 24: return launch_skinny_b<24>(p, nb, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace limb
}  // namespace ccm
