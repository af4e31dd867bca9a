// Dispatch of the Monte Carlo kernels (mc_kernel.hpp), and the reduction of their
// partials.
#include "dev.hpp"
#include "kernels.hpp"

namespace reach {

// One source each (mc_<system>_<type>.hip).
hipError_t launch_mc_ctm_f64(int mode, int E, const McArgs& a, hipStream_t s);
hipError_t launch_mc_ctm_f32(int mode, int E, const McArgs& a, hipStream_t s);
hipError_t launch_mc_rd_f64(int mode, int E, const McArgs& a, hipStream_t s);
hipError_t launch_mc_rd_f32(int mode, int E, const McArgs& a, hipStream_t s);
hipError_t launch_mc_lin3_f64(int mode, int E, const McArgs& a, hipStream_t s);
hipError_t launch_mc_lin3_f32(int mode, int E, const McArgs& a, hipStream_t s);

template <class T>
__device__ __forceinline__ T nan_min(T m, T x) {
    // NaN-propagating: once either side is NaN the result stays NaN.
    return (m != m) ? m : ((x < m || x != x) ? x : m);
}
template <class T>
__device__ __forceinline__ T nan_max(T m, T x) {
    return (m != m) ? m : ((x > m || x != x) ? x : m);
}

// Reduction of np partials lying wstep slots of `stride` values apart, in two
// launches when np > RED_CHUNK.  E > 0: a slot is one wave's [e][lane] block and
// block (e, g) owns its values [e][0..63] (cells j = lane * E + e); E = 0: a slot
// is the vector of n cells and block (b, g) owns cells 64 b .. 64 b + 63; of
// partials w in [g RED_CHUNK, (g + 1) RED_CHUNK): its RED_WAVES waves issue RED_CHUNK / RED_WAVES
// independent loads each, then combine through LDS.  The first launch writes
// each chunk's result over the chunk's first partial; the second (wstep times
// RED_CHUNK) reduces those and writes the box.  Min and max (NaN-propagating)
// are exact, so the split changes no value (signed zeros aside), and every
// block reads only its own chunk.
constexpr int RED_WAVES = 16;
constexpr int RED_CHUNK = 256;
constexpr int RED_PER_WAVE = RED_CHUNK / RED_WAVES;

template <class T>
__global__ __launch_bounds__(WAVE * RED_WAVES) void mc_reduce_kernel(
    T* __restrict__ pmin, T* __restrict__ pmax, int E, int64_t nw, int64_t wstep, int64_t n,
    T* __restrict__ rmin, T* __restrict__ rmax, unsigned int* status, int final_pass) {
    __shared__ T smin[RED_WAVES][WAVE];
    __shared__ T smax[RED_WAVES][WAVE];
    const int lane = threadIdx.x & (WAVE - 1);
    const int wv = threadIdx.x / WAVE;
    const int64_t j = E ? (int64_t)lane * E + blockIdx.x : (int64_t)blockIdx.x * WAVE + lane;
    // (an [e][lane] slot has room past cell n-1, a vector of cells has not)
    const size_t off = E || j < n ? (size_t)blockIdx.x * WAVE + (size_t)lane : 0;
    const size_t stride = E ? (size_t)E * WAVE : (size_t)n;
    const int64_t w0 = (int64_t)blockIdx.y * RED_CHUNK;
    const int64_t w1 = w0 + RED_CHUNK < nw ? w0 + RED_CHUNK : nw;
    // indices past the chunk load nothing and stand in with the identities
    // +inf / -inf (nan_min(x, +inf) = x for every x, NaN included; the
    // chunk's first partial always exists)
    T a[RED_PER_WAVE], b[RED_PER_WAVE];
#pragma unroll
    for (int u = 0; u < RED_PER_WAVE; ++u) {
        const int64_t w = w0 + wv + (int64_t)u * RED_WAVES;
        a[u] = T(__builtin_inf());
        b[u] = -T(__builtin_inf());
        if (w < w1) {   // the same in every lane of the wave
            const size_t idx = (size_t)(w * wstep) * stride + off;
            a[u] = pmin[idx];
            b[u] = pmax[idx];
        }
    }
    T mn = a[0], mx = b[0];
#pragma unroll
    for (int u = 1; u < RED_PER_WAVE; ++u) {
        mn = nan_min(mn, a[u]);
        mx = nan_max(mx, b[u]);
    }
    smin[wv][lane] = mn;
    smax[wv][lane] = mx;
    __syncthreads();
    if (wv != 0) return;
    mn = smin[0][lane];
    mx = smax[0][lane];
#pragma unroll
    for (int k = 1; k < RED_WAVES; ++k) {
        mn = nan_min(mn, smin[k][lane]);
        mx = nan_max(mx, smax[k][lane]);
    }
    if (!final_pass) {
        if (!E && j >= n) return;
        const size_t idx = (size_t)(w0 * wstep) * stride + off;
        pmin[idx] = mn;
        pmax[idx] = mx;
        return;
    }
    unsigned bits = 0;
    if (j < n) {
        rmin[j] = mn;
        rmax[j] = mx;
        if (!finiteT(mn) || !finiteT(mx)) bits = ST_NONFINITE;
    }
    report_status(status, bits);
}

hipError_t launch_mc(int kind, int mode, int dtype, int E, const McArgs& a, hipStream_t s) {
    const auto f = kind == K_CTM ? (dtype == 0 ? launch_mc_ctm_f64 : launch_mc_ctm_f32)
                 : kind == K_RD ? (dtype == 0 ? launch_mc_rd_f64 : launch_mc_rd_f32)
                 : kind == K_LIN3 ? (dtype == 0 ? launch_mc_lin3_f64 : launch_mc_lin3_f32)
                                  : nullptr;
    return f ? f(mode, E, a, s) : hipErrorInvalidValue;
}

bool mc_has_plain(int dtype, int E) {
    return E == 1 || E == 2 || E == 4 || E == 8 || E == 16 || E == 32 || (dtype == 1 && E == 64);
}
bool mc_has_segments(int dtype, int E) {
    return E == 1 || (E >= 2 && E <= 20 && E % 2 == 0) || E == 24 || E == 28 || E == 32 ||
           (dtype == 1 && (E == 40 || E == 48 || E == 56 || E == 60 || E == 64));
}
int mc_max_E(int dtype) { return dtype == 1 ? 64 : 32; }

template <class T>
static hipError_t reduce(int E, void* pmin, void* pmax, int64_t np, int64_t n, void* rmin,
                         void* rmax, unsigned int* status, hipStream_t s) {
    const dim3 block(WAVE * RED_WAVES);
    const unsigned cols = (unsigned)(E ? E : (n + WAVE - 1) / WAVE);
    const int64_t chunks = (np + RED_CHUNK - 1) / RED_CHUNK;
    if (chunks > 1) {
        hipLaunchKernelGGL((mc_reduce_kernel<T>), dim3(cols, (unsigned)chunks), block, 0, s,
                           (T*)pmin, (T*)pmax, E, np, 1, n, (T*)rmin, (T*)rmax, status, 0);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        static_assert(RED_CHUNK * RED_CHUNK >= kMcMaxWaves, "two passes cover every wave count");
        hipLaunchKernelGGL((mc_reduce_kernel<T>), dim3(cols, 1), block, 0, s, (T*)pmin, (T*)pmax,
                           E, chunks, (int64_t)RED_CHUNK, n, (T*)rmin, (T*)rmax, status, 1);
    } else {
        hipLaunchKernelGGL((mc_reduce_kernel<T>), dim3(cols, 1), block, 0, s, (T*)pmin, (T*)pmax,
                           E, np, 1, n, (T*)rmin, (T*)rmax, status, 1);
    }
    return hipGetLastError();
}

hipError_t launch_mc_reduce(int dtype, int E, void* pmin, void* pmax, int64_t np, int64_t n,
                            void* rmin, void* rmax, unsigned int* status, hipStream_t s) {
    return dtype == 0 ? reduce<double>(E, pmin, pmax, np, n, rmin, rmax, status, s)
                      : reduce<float>(E, pmin, pmax, np, n, rmin, rmax, status, s);
}

}  // namespace reach
