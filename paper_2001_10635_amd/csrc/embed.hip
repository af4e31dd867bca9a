// Dispatch of the embedding kernels (embed_tile.hpp) and the order check.
#include <algorithm>

#include "dev.hpp"
#include "kernels.hpp"

namespace reach {

// One source each (embed_<system>_<type>.hip).
hipError_t launch_embed_ctm_f64(int mode, int E, int S, bool pair, const EmbedPass& a,
                          int64_t grid, hipStream_t s);
hipError_t launch_embed_ctm_f32(int mode, int E, int S, bool pair, const EmbedPass& a,
                          int64_t grid, hipStream_t s);
hipError_t launch_embed_rd_f64(int mode, int E, int S, bool pair, const EmbedPass& a,
                          int64_t grid, hipStream_t s);
hipError_t launch_embed_rd_f32(int mode, int E, int S, bool pair, const EmbedPass& a,
                          int64_t grid, hipStream_t s);
hipError_t launch_embed_lin3_f64(int mode, int E, int S, bool pair, const EmbedPass& a,
                          int64_t grid, hipStream_t s);
hipError_t launch_embed_lin3_f32(int mode, int E, int S, bool pair, const EmbedPass& a,
                          int64_t grid, hipStream_t s);

// Lower > upper check of a finished box where no block sees both sides of a cell (the
// heat grid, and a last pass in blocks of one wave).
template <class T>
__global__ __launch_bounds__(256) void order_check_kernel(const T* __restrict__ lo,
                                                          const T* __restrict__ hi, int64_t n,
                                                          unsigned int* status) {
    unsigned bits = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        if (lo[i] > hi[i]) bits = ST_ORDER;
    report_status(status, bits);
}

bool embed_has_shape(int kind, int dtype, int E, int S) {
    const auto in = [E](std::initializer_list<int> es) {
        return std::find(es.begin(), es.end(), E) != es.end();
    };
    if (S == 2) return in({1, 2, 4, 6, 8, 12, 16}) || (dtype == 1 && E == 32);
    if (S == 1 && kind != K_LIN3)
        return in({1, 2, 4, 6, 8, 12, 16, 20, 24, 32}) || (dtype == 0 && E == 28) ||
               (dtype == 1 && (E == 48 || E == 64));
    return false;
}
int embed_max_E(int dtype, int S) {
    if (S == 1) return dtype == 1 ? 64 : 32;
    return dtype == 1 ? 32 : 16;
}

hipError_t launch_embed(int kind, int mode, int dtype, int E, int S, bool pair, EmbedPass a,
                        int64_t grid, hipStream_t s) {
    if (pair && S != 1) return hipErrorInvalidValue;
    if (kind == K_LIN3) a.alt = a.prm[2] < 0.0;   // the right coupling would cross the sides
    const auto f = kind == K_CTM ? (dtype == 0 ? launch_embed_ctm_f64 : launch_embed_ctm_f32)
                 : kind == K_RD ? (dtype == 0 ? launch_embed_rd_f64 : launch_embed_rd_f32)
                 : kind == K_LIN3 ? (dtype == 0 ? launch_embed_lin3_f64 : launch_embed_lin3_f32)
                                  : nullptr;
    return f ? f(mode, E, S, pair, a, grid, s) : hipErrorInvalidValue;
}

hipError_t launch_order_check(int dtype, const void* lo, const void* hi, int64_t n,
                              unsigned int* status, int64_t max_blocks, hipStream_t s) {
    const int64_t blocks = std::min<int64_t>((n + 255) / 256, max_blocks);
    if (dtype == 0)
        hipLaunchKernelGGL(order_check_kernel<double>, dim3((unsigned)blocks), dim3(256), 0, s,
                           (const double*)lo, (const double*)hi, n, status);
    else
        hipLaunchKernelGGL(order_check_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, s,
                           (const float*)lo, (const float*)hi, n, status);
    return hipGetLastError();
}

}  // namespace reach
