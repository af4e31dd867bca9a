// Embedding-system RK4 on gfx950: the mixed-monotonicity method of PIRK
// (Sec. 2.1; Algorithm 3 with Algorithm 1 as integrator), fused and
// temporally blocked.
//
// One wavefront owns a window of 64*E cells of both the lower and the upper
// vector (E cells per lane, both sides in the same lane so the coupled LIN3
// decomposition function sees x and xh of its neighbours).  A pass loads the
// window once, runs `ksteps` RK4 steps entirely in registers (four stages per
// step, neighbour values by DPP lane shifts), and writes back only the cells
// that are still exact: each stage lets a cut window edge corrupt one more
// cell, so a pass of K steps keeps a halo of H = 4K cells per cut edge.
// Windows that start at cell 0 or reach cell n-1 use the chain's own boundary
// conditions there and lose nothing on that side.  HBM traffic is one read
// and one write of 2n values per pass, i.e. per K steps.
//
// Global <-> register transfers go through LDS (tile_io.hpp).
//
// The kernel template; one source per system and type instantiates it
// (embed_*.hip), embed.hip holds the dispatch.
#pragma once
#include "kernels.hpp"
#include "tile_io.hpp"

namespace reach {

// S = 2: a wave holds both sides of its window (any system, including the
// coupled LIN3).  S = 1: a wave holds one side (cooperative systems only, whose
// decomposition function reads one side), so the same registers cover twice
// the cells and the halo share halves; tiles [0, W) are the lower side and
// [W, 2W) the upper side.  PAIR (S = 1): a block of two waves, the lower and the
// upper side of one window.  The call's last pass runs so: the upper wave hands
// its box to the lower one through LDS, which compares them, where a separate
// kernel would read both results again (1 GiB at 2^26 cells); every pass of a
// single window runs so too.
//
// LIN3 runs as K_LIN3C or K_LIN3M: with the sign of each coupling known its
// decomposition function has 4 nonzero terms of 7.  Exchanging the two sides of
// every odd cell (a.alt) turns a coupling that crosses the sides into one that
// does not and the reverse, so that the right one never crosses (for E > 1 a
// lane's first cell has the parity of the window's).  The
// terms left out are zero coefficients times values: they change a result only
// where that value is not finite (0 times inf is NaN).  A window that ends with
// a non-finite value is therefore run again from its input with every term
// (such a value never turns finite again, so a window without one is exact).
//
// One side of up to 192 bytes a lane keeps to 256 registers (two waves per SIMD;
// per-cell inputs would take 2 to 10 more).
template <int KIND, class T, int E, int MODE, int S, bool PAIR>
__global__ __launch_bounds__(PAIR ? 2 * WAVE : WAVE, S == 1 && E * sizeof(T) <= 192 ? 2 : 1)
void embed_tile_kernel(EmbedPass a) {
    using IO = TileIO<T, E>;
    constexpr bool LIN = KIND == K_LIN3C || KIND == K_LIN3M;
    // one wave's staging rows; in a pair also the box the upper wave hands over
    constexpr int ROW = IO::STAGED ? IO::ROW : E;
    constexpr int LDS = IO::STAGED || !PAIR ? IO::LDS_ELEMS : WAVE * E;
    __shared__ __attribute__((aligned(16))) T lds[LDS * (PAIR ? 2 : 1)];
    const int lane = threadIdx.x & (WAVE - 1);

    // blockIdx -> tile: consecutive tiles on one XCD share halos in its L2.
    const int64_t b = blockIdx.x;
    int64_t g = (b & 7) * (int64_t)a.per_xcd + (b >> 3);
    if (g >= (S == 1 && !PAIR ? 2 * a.W : a.W)) return;
    const int side = PAIR ? (int)(threadIdx.x / WAVE) : (S == 1 && g >= a.W) ? 1 : 0;
    T* const my_lds = lds + (PAIR ? side * LDS : 0);
    const int64_t w = PAIR ? g : g - side * a.W;

    // the last of several windows ends with the chain instead of running past
    // it (a window that holds padding pays a select per cell and stage, 1.3 x
    // the instructions, and a launch of few waves waits for that one); it owns
    // the cells the window before it could not finish
    const int64_t span = (int64_t)WAVE * E;
    const bool last = w == a.W - 1;
    const int64_t ts = last && w > 0 ? a.n - span : w * a.OUT;
    const bool reaches_end = ts + span >= a.n;
    const bool fast = ts + span <= a.n;
    const T* src[2] = {(const T*)a.src_lo, (const T*)a.src_hi};
    T* dst[2] = {(T*)a.dst_lo, (T*)a.dst_hi};
    const T* pin[2] = {(const T*)a.p_lo, (const T*)a.p_hi};

    T y[S][E];
#pragma unroll
    for (int s = 0; s < S; ++s)
        IO::load(y[s], src[S == 1 ? side : s], ts, a.n, ghost<KIND, T>(), fast, a.nt, my_lds);

    Inputs<T, E, S, MODE> U;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const T* p = pin[S == 1 ? side : s];
        if constexpr (MODE == IN_SCALAR) {
            U.u[s] = p ? p[0] : T(0);
        } else if constexpr (MODE == IN_ALT) {
            U.u[s][0] = U.u[s][1] = p ? p[0] : T(0);
        } else {
            IO::load(U.u[s], p, ts, a.n, T(0), fast, false, my_lds);
        }
    }
    // A single window may write its results over its inputs, also one side's over
    // the other's: both waves have read before either writes.  (Several windows
    // never write what a pass reads.)
    if constexpr (PAIR) {
        if (a.W == 1) __syncthreads();
    }
    const SysPrm<T> P = make_prm<T>(a.prm);
    const Steps<T> st = {(T)a.h2, (T)a.dt, (T)a.dt6};

    // the sides of the odd cells exchanged (state; inputs: see below)
    [[maybe_unused]] const int odd0 = (int)(ts & 1) ^ (E == 1 ? (lane & 1) : 0);
    [[maybe_unused]] const auto exchange = [&](auto& v0, auto& v1, int len) {
#pragma unroll
        for (int e = 0; e < len; ++e) {
            const bool sw = ((E == 1 ? 0 : e & 1) ^ odd0) != 0;
            const T p = v0[e], q = v1[e];
            v0[e] = sw ? q : p;
            v1[e] = sw ? p : q;
        }
    };

    // cells of this lane inside the chain (the others hold the ghost)
    const int64_t left = a.n - (ts + (int64_t)lane * E);
    const int nvalid = (int)(left < 0 ? 0 : (left > E ? E : left));
    if constexpr (!LIN) {
        if (fast) {
            // no cell is padding; for the CTM lane 63's right neighbour is the
            // ghost where the window ends the chain
            if (KIND == K_CTM && reaches_end) {
                Mask<E, false, true> M{E};
                rk4_steps<KIND, T, E, S, MODE>(y, a.ksteps, P, U, st, M);
            } else {
                Mask<E, false, false> M{E};
                rk4_steps<KIND, T, E, S, MODE>(y, a.ksteps, P, U, st, M);
            }
        } else if constexpr (S == 1) {
            // a single window, longer than the chain: one indexed move a stage
            // sets the ghost, cheaper than the selects from 48 bytes a lane on (400
            // steps of 500 cells: FP64 CTM 236 -> 208 us, RD 194 -> 182; FP32, 32
            // bytes, 157 -> 192)
            const auto M = chain_end_mask<E, true, (E * sizeof(T) >= 48)>(a.n - ts);
            rk4_steps<KIND, T, E, S, MODE>(y, a.ksteps, P, U, st, M);
        } else {
            Mask<E, true, true> M{nvalid};
            rk4_steps<KIND, T, E, S, MODE>(y, a.ksteps, P, U, st, M);
        }
    } else {
        Inputs<T, E, S, MODE> V = U;   // the input each side of a cell takes
        constexpr int NU = MODE == IN_CELL ? E : 2;
        if (P.a3 < T(0)) {             // b < 0: d falls with the other side's input
#pragma unroll
            for (int e = 0; e < NU; ++e) {
                V.u[0][e] = U.u[1][e];
                V.u[1][e] = U.u[0][e];
            }
        }
        if (a.alt) {
            exchange(y[0], y[1], E);
            exchange(V.u[0], V.u[1], NU);
        }
        if (fast) {
            Mask<E, false, false> M{E};
            rk4_steps<KIND, T, E, S, MODE>(y, a.ksteps, P, V, st, M);
        } else {
            Mask<E, true, true> M{nvalid};
            rk4_steps<KIND, T, E, S, MODE>(y, a.ksteps, P, V, st, M);
        }
        bool finite = true;
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int e = 0; e < E; ++e) finite = finite && finiteT(y[s][e]);
        if (__any(!finite)) {
#pragma unroll
            for (int s = 0; s < S; ++s) {
                IO::load(y[s], src[s], ts, a.n, T(0), fast, false, my_lds);
                if constexpr (MODE == IN_CELL)
                    IO::load(U.u[s], pin[s], ts, a.n, T(0), fast, false, my_lds);
            }
            Mask<E, true, true> M{nvalid};
            rk4_steps<K_LIN3, T, E, S, MODE>(y, a.ksteps, P, U, st, M);
        } else if (a.alt) {
            exchange(y[0], y[1], E);
        }
    }

    const int olo = (w == 0) ? 0 : a.H + (int)(w * a.OUT - ts);
    const int ohi = reaches_end ? (int)(a.n - ts) : (int)(span - a.H);
#pragma unroll
    for (int s = 0; s < S; ++s)
        IO::store(y[s], dst[S == 1 ? side : s], ts, olo, ohi, fast, a.nt, my_lds);

    if (a.check) {
        unsigned bits = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int el = lane * E + e;
            if (el >= olo && el < ohi) {
#pragma unroll
                for (int s = 0; s < S; ++s)
                    if (!finiteT(y[s][e])) bits |= ST_NONFINITE;
                if constexpr (S == 2) {
                    if (y[0][e] > y[1][e]) bits |= ST_ORDER;
                }
            }
        }
        if constexpr (PAIR) {
            // the upper wave hands its box to the lower one
            T* const upper = lds + LDS;
            if (side == 1) {
#pragma unroll
                for (int e = 0; e < E; ++e) upper[lane * ROW + e] = y[0][e];
            }
            __syncthreads();
            if (side == 0) {
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int el = lane * E + e;
                    if (el >= olo && el < ohi && y[0][e] > upper[lane * ROW + e]) bits |= ST_ORDER;
                }
            }
        }
        report_status(a.status, bits);
    }
}

template <int KIND, class T, int E, int MODE, int S, bool PAIR = false>
static hipError_t go(const EmbedPass& a, int64_t grid, hipStream_t s) {
    hipLaunchKernelGGL((embed_tile_kernel<KIND, T, E, MODE, S, PAIR>), dim3((unsigned)grid),
                       dim3(PAIR ? 2 * WAVE : WAVE), 0, s, a);
    return hipGetLastError();
}
template <int KIND, class T, int E, int MODE>
static hipError_t go_one_side(bool pair, const EmbedPass& a, int64_t grid, hipStream_t s) {
    return pair ? go<KIND, T, E, MODE, 1, true>(a, grid, s) : go<KIND, T, E, MODE, 1, false>(a, grid, s);
}

// Shapes built: S = 2 (both sides per wave) for every system, S = 1 (one side
// per wave, wider tiles) for the cooperative CTM and RD chains.
template <int KIND, class T, int MODE>
static hipError_t by_E(int E, int S, bool pair, const EmbedPass& a, int64_t grid, hipStream_t s) {
    constexpr bool F32 = sizeof(T) == 4;
    constexpr bool COOP = KIND == K_CTM || KIND == K_RD;
    if (S == 2) {
        switch (E) {
            case 1: return go<KIND, T, 1, MODE, 2>(a, grid, s);
            case 2: return go<KIND, T, 2, MODE, 2>(a, grid, s);
            case 4: return go<KIND, T, 4, MODE, 2>(a, grid, s);
            case 6: return go<KIND, T, 6, MODE, 2>(a, grid, s);
            case 8: return go<KIND, T, 8, MODE, 2>(a, grid, s);
            case 12: return go<KIND, T, 12, MODE, 2>(a, grid, s);
            case 16: return go<KIND, T, 16, MODE, 2>(a, grid, s);
            case 32:
                if constexpr (F32) return go<KIND, T, 32, MODE, 2>(a, grid, s);
                else return hipErrorInvalidValue;
            default: return hipErrorInvalidValue;
        }
    }
    if constexpr (COOP) {
        if (S == 1) {
            switch (E) {
                case 1: return go_one_side<KIND, T, 1, MODE>(pair, a, grid, s);
                case 2: return go_one_side<KIND, T, 2, MODE>(pair, a, grid, s);
                case 4: return go_one_side<KIND, T, 4, MODE>(pair, a, grid, s);
                case 6: return go_one_side<KIND, T, 6, MODE>(pair, a, grid, s);
                case 8: return go_one_side<KIND, T, 8, MODE>(pair, a, grid, s);
                case 12: return go_one_side<KIND, T, 12, MODE>(pair, a, grid, s);
                case 16: return go_one_side<KIND, T, 16, MODE>(pair, a, grid, s);
                case 20: return go_one_side<KIND, T, 20, MODE>(pair, a, grid, s);
                case 24: return go_one_side<KIND, T, 24, MODE>(pair, a, grid, s);
                case 28:   // FP64: the widest one-side tile within 256 VGPRs
                    if constexpr (!F32) return go_one_side<KIND, T, 28, MODE>(pair, a, grid, s);
                    else return hipErrorInvalidValue;
                case 32: return go_one_side<KIND, T, 32, MODE>(pair, a, grid, s);
                case 48:
                    if constexpr (F32) return go_one_side<KIND, T, 48, MODE>(pair, a, grid, s);
                    else return hipErrorInvalidValue;
                case 64:
                    if constexpr (F32) return go_one_side<KIND, T, 64, MODE>(pair, a, grid, s);
                    else return hipErrorInvalidValue;
                default: return hipErrorInvalidValue;
            }
        }
    }
    return hipErrorInvalidValue;
}

}  // namespace reach
