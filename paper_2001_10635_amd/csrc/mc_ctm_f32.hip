// Monte Carlo kernels of the CTM chain in FP32 (see mc_kernel.hpp).
#include "mc_kernel.hpp"

namespace reach {

hipError_t launch_mc_ctm_f32(int, int E, const McArgs& a, hipStream_t s) {
    return by_E<K_CTM, float, IN_SCALAR>(E, a, s);
}

}  // namespace reach
