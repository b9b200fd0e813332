// The limb GEMM for operands A of 2 limb(s) (see gemm_limb.hpp).
#include "gemm_limb_impl.hpp"

namespace ccm {
namespace limb {

hipError_t launch_pass_a2(const GemmArgs &p, int lb, int out32, hipStream_t s) {
  return launch_pass_la<2>(p, lb, out32, s);
}

}  // namespace limb
}  // namespace ccm
