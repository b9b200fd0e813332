// The narrow-B product for A of 9 to 16 bits (see gemm_skinny.hpp).
#include "gemm_skinny.hpp"

namespace ccm {
namespace limb {

hipError_t launch_skinny_2(const SkinnyArgs &p, int abits, int nb, hipStream_t s) {
  switch (abits) {
    case 9: return launch_skinny_b<9>(p, nb, s);
    case 10: return launch_skinny_b<10>(p, nb, s);
    case 11: return launch_skinny_b<11>(p, nb, s);
    case 12: return launch_skinny_b<12>(p, nb, s);
    case 13: return launch_skinny_b<13>(p, nb, s);
    case 14: return launch_skinny_b<14>(p, nb, s);
    case 15: return launch_skinny_b<15>(p, nb, s);
    case 16: return launch_skinny_b<16>(p, nb, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace limb
}  // namespace ccm
