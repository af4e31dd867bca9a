// Monte Carlo kernels of the LIN3 chain in FP64 (see mc_kernel.hpp).
#include "mc_kernel.hpp"

namespace reach {

hipError_t launch_mc_lin3_f64(int mode, int E, const McArgs& a, hipStream_t s) {
    return mode ? by_E<K_LIN3, double, IN_CELL>(E, a, s) : by_E<K_LIN3, double, IN_SCALAR>(E, a, s);
}

}  // namespace reach
