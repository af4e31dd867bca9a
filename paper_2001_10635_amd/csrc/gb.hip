// Contraction / growth-bound reachable box on gfx950 (PIRK Sec. 2.1,
// Algorithm 2).
//
// Two RK4 runs share every launch: one wave integrates the center
// of the box with the system's own f at the center input, another the
// half-width of the same window with the linear growth dynamics
// r' = C r + |b| [p], C the tridiagonal contraction matrix.  Each wave holds one
// run's window in registers, exactly like the one-side embedding tiles (same
// per-cell code, transfers, temporal blocking and halos).  The first pass forms
// c = (lo + hi) / 2 or r = (hi - lo) / 2 as it loads the box.  The two waves of a
// window are one block (PAIR); in the last pass they exchange their windows through
// LDS and write [c - r, c + r] themselves: a separate combining kernel reads c and r
// and writes the box again, 64 bytes per FP64 cell.  It remains for calls whose result
// arrays overlap what the last pass still reads, and for a last pass whose waves are
// blocks of their own because blocks of two would share SIMDs (pairs_share in the
// runtime has the figures).
#include <algorithm>

#include "kernels.hpp"
#include "tile_io.hpp"

namespace reach {

template <int KIND, class T, int E, int MODE, bool PAIR>
__global__ __launch_bounds__(PAIR ? 2 * WAVE : WAVE, E * sizeof(T) <= 192 ? 2 : 1)
void gb_tile_kernel(GbPass a) {
    using IO = TileIO<T, E>;
    constexpr int ROW = IO::STAGED ? IO::ROW : E;
    constexpr int LDS = IO::STAGED || !PAIR ? IO::LDS_ELEMS : WAVE * E;
    __shared__ __attribute__((aligned(16))) T lds[LDS * (PAIR ? 2 : 1)];
    const int lane = threadIdx.x & (WAVE - 1);
    const int64_t b = blockIdx.x;
    const int64_t g = (b & 7) * (int64_t)a.per_xcd + (b >> 3);
    if (g >= (PAIR ? a.W : 2 * a.W)) return;
    // 0: center run, 1: half-width run
    const int side = PAIR ? (int)(threadIdx.x / WAVE) : g >= a.W ? 1 : 0;
    const int64_t w = PAIR ? g : g - side * a.W;
    T* const my_lds = lds + (PAIR ? side * LDS : 0);
    // the last of several windows ends with the chain (see embed_tile_kernel)
    const int64_t span = (int64_t)WAVE * E;
    const int64_t ts = w == a.W - 1 && w > 0 ? a.n - span : w * a.OUT;
    const bool reaches_end = ts + span >= a.n;
    const bool fast = !PAIR || ts + span <= a.n;   // (only a single window holds padding)
    const int64_t left = a.n - (ts + (int64_t)lane * E);
    const int nvalid = (int)(left < 0 ? 0 : (left > E ? E : left));

    // center p = (lo + hi) / 2 or half-width (hi - lo) / 2 of an interval
    const auto part = [side](T lo, T hi) { return side == 0 ? (lo + hi) / T(2) : (hi - lo) / T(2); };
    const T out = side == 0 ? ghost<KIND, T>() : T(0);   // cells past the chain
    T y[1][E];
    if (a.first) {
        T hi[E];
        IO::load(y[0], (const T*)a.x_lo, ts, a.n, T(0), fast, false, my_lds);
        IO::load(hi, (const T*)a.x_hi, ts, a.n, T(0), fast, false, my_lds);
#pragma unroll
        for (int e = 0; e < E; ++e) y[0][e] = e < nvalid ? part(y[0][e], hi[e]) : out;
    } else {
        IO::load(y[0], (const T*)(side == 0 ? a.src_c : a.src_r), ts, a.n, out, fast, false, my_lds);
    }

    Inputs<T, E, 1, MODE> U;
    const T* pl = (const T*)a.p_lo;
    const T* ph = (const T*)a.p_hi;
    if constexpr (MODE == IN_SCALAR) {
        U.u[0] = pl ? part(pl[0], ph[0]) : T(0);
    } else {
        T hi[E];
        IO::load(U.u[0], pl, ts, a.n, T(0), fast, false, my_lds);
        IO::load(hi, ph, ts, a.n, T(0), fast, false, my_lds);
#pragma unroll
        for (int e = 0; e < E; ++e) U.u[0][e] = part(U.u[0][e], hi[e]);
    }
    const Steps<T> st = {(T)a.h2, (T)a.dt, (T)a.dt6};
    const SysPrm<T> P = make_prm<T>(side == 0 ? a.prm : a.prm_r);

    const Mask<E, false, false> inner{E};
    const Mask<E, false, true> end{E};
    const auto padded = chain_end_mask<E, true, (E * sizeof(T) >= 48)>(a.n - ts);
    if (side == 0) {
        if (!fast) rk4_steps<KIND, T, E, 1, MODE>(y, a.ksteps, P, U, st, padded);
        else if (KIND == K_CTM && reaches_end) rk4_steps<KIND, T, E, 1, MODE>(y, a.ksteps, P, U, st, end);
        else rk4_steps<KIND, T, E, 1, MODE>(y, a.ksteps, P, U, st, inner);
    } else {
        if (!fast) rk4_steps<K_LIN3, T, E, 1, MODE>(y, a.ksteps, P, U, st, padded);
        else rk4_steps<K_LIN3, T, E, 1, MODE>(y, a.ksteps, P, U, st, inner);
    }

    const int olo = (w == 0) ? 0 : a.H + (int)(w * a.OUT - ts);
    const int ohi = reaches_end ? (int)(a.n - ts) : (int)(span - a.H);
    if (!PAIR || !a.last) {
        IO::store(y[0], (T*)(side == 0 ? a.dst_c : a.dst_r), ts, olo, ohi, fast, false, my_lds);
        return;
    }
    if constexpr (PAIR) {
        // [c - r, c + r]: the center wave writes the lower vector, the other the upper
#pragma unroll
        for (int e = 0; e < E; ++e) my_lds[lane * ROW + e] = y[0][e];
        __syncthreads();
        const T* const other = lds + (1 - side) * LDS;
        unsigned bits = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const T o = other[lane * ROW + e];
            const T c = side == 0 ? y[0][e] : o, r = side == 0 ? o : y[0][e];
            const T lo = c - r, hi = c + r;
            const int el = lane * E + e;
            if (el >= olo && el < ohi) {
                if (!finiteT(lo) || !finiteT(hi)) bits |= ST_NONFINITE;
                if (lo > hi) bits |= ST_ORDER;
            }
            y[0][e] = side == 0 ? lo : hi;
        }
        __syncthreads();   // both have read before the rows stage the stores
        IO::store(y[0], (T*)(side == 0 ? a.r_lo : a.r_hi), ts, olo, ohi, fast, false, my_lds);
        report_status(a.status, bits);
    }
}

template <class T>
__global__ __launch_bounds__(256) void gb_combine_kernel(const T* __restrict__ c,
                                                         const T* __restrict__ r, int64_t n,
                                                         T* __restrict__ lo, T* __restrict__ hi,
                                                         unsigned int* status) {
    unsigned bits = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const T l = c[i] - r[i], h = c[i] + r[i];
        lo[i] = l;
        hi[i] = h;
        if (!finiteT(l) || !finiteT(h)) bits |= ST_NONFINITE;
        if (l > h) bits |= ST_ORDER;
    }
    report_status(status, bits);
}

template <int KIND, class T, int E, int MODE>
static hipError_t go_gb(const GbPass& a, int64_t grid, hipStream_t s) {
    if (a.pair)
        hipLaunchKernelGGL((gb_tile_kernel<KIND, T, E, MODE, true>), dim3((unsigned)grid),
                           dim3(2 * WAVE), 0, s, a);
    else
        hipLaunchKernelGGL((gb_tile_kernel<KIND, T, E, MODE, false>), dim3((unsigned)grid),
                           dim3(WAVE), 0, s, a);
    return hipGetLastError();
}

template <int KIND, class T, int MODE>
static hipError_t gb_by_E(int E, const GbPass& a, int64_t grid, hipStream_t s) {
    switch (E) {
        case 1: return go_gb<KIND, T, 1, MODE>(a, grid, s);
        case 2: return go_gb<KIND, T, 2, MODE>(a, grid, s);
        case 4: return go_gb<KIND, T, 4, MODE>(a, grid, s);
        case 8: return go_gb<KIND, T, 8, MODE>(a, grid, s);
        case 12: return go_gb<KIND, T, 12, MODE>(a, grid, s);
        case 16: return go_gb<KIND, T, 16, MODE>(a, grid, s);
        case 20: return go_gb<KIND, T, 20, MODE>(a, grid, s);
        case 24: return go_gb<KIND, T, 24, MODE>(a, grid, s);
        case 28: return go_gb<KIND, T, 28, MODE>(a, grid, s);
        case 32: return go_gb<KIND, T, 32, MODE>(a, grid, s);
        default: return hipErrorInvalidValue;
    }
}

bool gb_has_E(int E) {
    return E == 1 || E == 2 || E == 4 || E == 8 || E == 12 || E == 16 || E == 20 || E == 24 ||
           E == 28 || E == 32;
}

hipError_t launch_gb(int kind, int mode, int dtype, int E, GbPass a, hipStream_t s) {
    const int64_t blocks = a.pair ? a.W : 2 * a.W;
    a.per_xcd = (int32_t)((blocks + 7) / 8);
    const int64_t grid = 8 * (int64_t)a.per_xcd;
    if (dtype == 0) {
        if (kind == K_CTM) return gb_by_E<K_CTM, double, IN_SCALAR>(E, a, grid, s);
        if (kind == K_RD) return mode ? gb_by_E<K_RD, double, IN_CELL>(E, a, grid, s)
                                      : gb_by_E<K_RD, double, IN_SCALAR>(E, a, grid, s);
        if (kind == K_LIN3) return mode ? gb_by_E<K_LIN3, double, IN_CELL>(E, a, grid, s)
                                        : gb_by_E<K_LIN3, double, IN_SCALAR>(E, a, grid, s);
    } else {
        if (kind == K_CTM) return gb_by_E<K_CTM, float, IN_SCALAR>(E, a, grid, s);
        if (kind == K_RD) return mode ? gb_by_E<K_RD, float, IN_CELL>(E, a, grid, s)
                                      : gb_by_E<K_RD, float, IN_SCALAR>(E, a, grid, s);
        if (kind == K_LIN3) return mode ? gb_by_E<K_LIN3, float, IN_CELL>(E, a, grid, s)
                                        : gb_by_E<K_LIN3, float, IN_SCALAR>(E, a, grid, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_gb_combine(int dtype, const void* c, const void* r, int64_t n, void* lo,
                             void* hi, unsigned int* status, int64_t max_blocks, hipStream_t s) {
    const int64_t blocks = std::min<int64_t>((n + 255) / 256, max_blocks);
    if (dtype == 0)
        hipLaunchKernelGGL(gb_combine_kernel<double>, dim3((unsigned)blocks), dim3(256), 0, s,
                           (const double*)c, (const double*)r, n, (double*)lo, (double*)hi, status);
    else
        hipLaunchKernelGGL(gb_combine_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, s,
                           (const float*)c, (const float*)r, n, (float*)lo, (float*)hi, status);
    return hipGetLastError();
}

}  // namespace reach
