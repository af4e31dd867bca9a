// Monte Carlo kernels of the RD chain in FP32 (see mc_kernel.hpp).
#include "mc_kernel.hpp"

namespace reach {

hipError_t launch_mc_rd_f32(int mode, int E, const McArgs& a, hipStream_t s) {
    return mode ? by_E<K_RD, float, IN_CELL>(E, a, s) : by_E<K_RD, float, IN_SCALAR>(E, a, s);
}

}  // namespace reach
