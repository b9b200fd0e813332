// The limb GEMM for operands A of three or four limbs (see gemm_limb.hpp).
#include "gemm_limb_impl.hpp"

namespace ccm {
namespace limb {

hipError_t launch_pass_a3(const GemmArgs &p, int lb, int out32, hipStream_t s) {
  return launch_pass_la<3>(p, lb, out32, s);
}

hipError_t launch_pass_a4(const GemmArgs &p, int lb, int out32, hipStream_t s) {
  return launch_pass_la<4>(p, lb, out32, s);
}

}  // namespace limb
}  // namespace ccm
