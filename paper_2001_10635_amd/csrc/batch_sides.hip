// Packed batches whose longest items run one side per wave (see batch.hip).
#include "batch_pack.hpp"

namespace reach {

hipError_t launch_pack_sides(const QDesc* d, const BatchItem* items, const uint32_t* members,
                             const uint64_t* n_items, unsigned long long* counter,
                             unsigned int* qflags, unsigned int* pair, unsigned int* status,
                             bool wide, int64_t grid, hipStream_t s) {
    if (wide)
        hipLaunchKernelGGL(pack_sides_kernel<16>, dim3((unsigned)grid), dim3(WAVE), 0, s, d, items,
                           members, n_items, counter, qflags, pair, status);
    else
        hipLaunchKernelGGL(pack_sides_kernel<8>, dim3((unsigned)grid), dim3(WAVE), 0, s, d, items,
                           members, n_items, counter, qflags, pair, status);
    return hipGetLastError();
}

}  // namespace reach
