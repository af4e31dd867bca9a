// Monte Carlo reachable box on gfx950 (PIRK Sec. 2.1, Algorithm 4).
//
// Each wavefront integrates whole samples: the full n-cell state of a sample
// lives in the wave's registers, so a sample's N RK4 steps touch no memory at
// all.  Waves (four per workgroup) are persistent: wave w takes sample groups
// w, w + nw, ... and folds each final state into a running min / max the
// workgroup keeps in LDS (one integer atomic per value: the running values are
// order-preserving integers, so min and max are exact in any order, NaN
// included).  At the end a workgroup writes its min / max, and a second kernel
// reduces those ceil(nw / 4) partials per dimension.
//
// Two layouts:
//   plain    E cells in each of the 64 lanes, n = 64 E (or, at the widest lanes
//            only, fewer with a select per cell);
//   segments the sample fills L = ceil(n / E) lanes, the first F = n - L (E - 1)
//            of them with E cells and the others ("short" lanes) with E - 1, so
//            that cell n-1 is the last cell of lane L-1 and no cell has a padded
//            neighbour inside its lane; 64 / L samples share the wave.  Per
//            stage a short lane takes its last cell's right neighbour, and the
//            value it hands to its right, by a select, and a sample's first and
//            last lanes their boundary values: a few selects per stage and
//            lane, none per cell.
// The host picks E and the layout by the instructions a sample costs (see
// mc_plan): a long chain the narrowest lanes that hold it, a short one with
// many samples several samples to a wave.
//
// Sampling: x0_j = x_lo_j + U(s, j) (x_hi_j - x_lo_j) and, for inputs,
// p_k = p_lo_k + U(s, n + k) (p_hi_k - p_lo_k), with U(s, j) word j mod 4 of
// Philox4x64-10 at key (seed, 0), counter (floor(j/4), s, 2, 0): counter-based,
// so any sample can be drawn independently and sample ranges compose.
//
// The kernel template; one source per system and type instantiates it
// (mc_*.hip), mc.hip holds the dispatch and the reduction.
#pragma once
#include "dev.hpp"
#include "kernels.hpp"

namespace reach {

// Waves per workgroup.  Each wave is independent; grouping four makes the
// dispatcher give a small launch (a few hundred samples) one wave per SIMD
// instead of stacking single-wave groups on the same SIMDs.
constexpr int MC_WPB = kMcWavesPerGroup;

// Order-preserving integers: a < b as floats iff key(a) < key(b).  NaN gets the
// key that wins the min (0) or the max (all ones), so it stays.
template <class T> struct Key;
template <> struct Key<float> {
    using U = unsigned int;
    static constexpr U TOP = 0x80000000u;
    static __device__ __forceinline__ U bits(float x) { return __float_as_uint(x); }
    static __device__ __forceinline__ float from(U u) { return __uint_as_float(u); }
};
template <> struct Key<double> {
    using U = unsigned long long;
    static constexpr U TOP = 0x8000000000000000ull;
    static __device__ __forceinline__ U bits(double x) { return (U)__double_as_longlong(x); }
    static __device__ __forceinline__ double from(U u) { return __longlong_as_double((long long)u); }
};
template <class T> __device__ __forceinline__ typename Key<T>::U to_key(T x) {
    const auto u = Key<T>::bits(x);
    return (u & Key<T>::TOP) ? ~u : (u | Key<T>::TOP);
}
template <class T> __device__ __forceinline__ T from_key(typename Key<T>::U k) {
    if (k == 0 || k == ~(typename Key<T>::U)0) return T(__builtin_nan(""));
    return Key<T>::from((k & Key<T>::TOP) ? (k & ~Key<T>::TOP) : ~k);
}

// Draws U(s, first .. first + E - 1) and hands each to f(e, u): one Philox block
// per four coordinates.  ZERO: first is a multiple of 4 in every lane; else the
// offset into the first block differs from lane to lane and the words are
// picked by selects.  The groups are kept apart (the compiler moves no memory
// access across the empty asm and nothing across the scheduling barrier), so
// that their loads and blocks do not pile up in registers that the step loop
// would pay for in waves per SIMD (CTM FP32, 64 cells a lane: 454 registers
// without).
template <class T, int E, bool ZERO, class F>
__device__ __forceinline__ void mc_draw(int64_t first, uint64_t s, uint64_t seed, F&& f) {
    const int64_t b0 = first >> 2;
    const int o = (int)(first & 3);
    U4 cur = philox4x64_10((uint64_t)b0, s, MC_STREAM, 0, seed, 0);
#pragma unroll
    for (int g = 0; g < (E + 3) / 4; ++g) {
        U4 nxt = cur;
        if ((ZERO && 4 * g + 4 < E) || (!ZERO && E > 1))
            nxt = philox4x64_10((uint64_t)(b0 + g + 1), s, MC_STREAM, 0, seed, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (4 * g + q >= E) continue;
            uint64_t word = cur.x[q];
            if constexpr (!ZERO) {
                const uint64_t w1 = q + 1 < 4 ? cur.x[(q + 1) & 3] : nxt.x[(q + 1) & 3];
                const uint64_t w2 = q + 2 < 4 ? cur.x[(q + 2) & 3] : nxt.x[(q + 2) & 3];
                const uint64_t w3 = q + 3 < 4 ? cur.x[(q + 3) & 3] : nxt.x[(q + 3) & 3];
                word = o == 0 ? word : o == 1 ? w1 : o == 2 ? w2 : w3;
            }
            f(4 * g + q, unif(word, T(0)));
        }
        cur = nxt;
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    }
}

// A lane of the segment layout.
struct Seg {
    bool shortl;   // holds E - 1 cells
    bool begin;    // holds cell 0 of its sample
    bool end;      // holds cell n-1
};

template <int E, class T>
__device__ __forceinline__ T seg_right(const T (&in)[E], int e, T rn, bool shortl) {
    if (e == E - 1) return rn;
    if (e == E - 2) return shortl ? rn : in[E - 1];
    return in[e + 1];
}
template <int E, class T>
__device__ __forceinline__ T seg_last(const T (&in)[E], bool shortl) {
    return E > 1 && shortl ? in[E > 1 ? E - 2 : 0] : in[E - 1];
}

// One RK4 stage in the segment layout; per cell the arithmetic is rk_stage's.
template <int KIND, int STAGE, class T, int E, int MODE>
__device__ __forceinline__ void seg_stage(T (&y)[E], T (&acc)[E], T (&t)[E], const SysPrm<T>& P,
                                          const Inputs<T, E, 1, MODE>& U, const Steps<T>& st,
                                          const Seg& L) {
    T (&in)[E] = (STAGE == 1) ? y : t;
    if constexpr (KIND == K_CTM) {
        // free outflow past cell n-1 (ghost -inf), zero inflow into cell 0
        const T v = P.a0, w = P.a1, wc = P.a2, q = P.a3;
        T rn = from_right(in[0]);
        rn = L.end ? neg_inf<T>() : rn;
        const auto flux = [&](int e) {
            return minT(minT(v * in[e], fmaT(-w, seg_right<E>(in, e, rn, L.shortl), wc)), q);
        };
        // the fluxes out of the lane's last two slots, one of which the next lane
        // takes, before any cell is updated
        const T FE = flux(E - 1), FD = E > 1 ? flux(E > 1 ? E - 2 : 0) : FE;
        T Fprev = from_left(L.shortl ? FD : FE);
        Fprev = L.begin ? T(0) : Fprev;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const T F = e == E - 1 ? FE : e == E - 2 ? FD : flux(e);
            const T k = Fprev - F;
            Fprev = F;
            rk_update<STAGE>(k, y[e], acc[e], t[e], st);
        }
    } else {
        // ghosts 0
        T left = from_left(seg_last<E>(in, L.shortl));
        T rn = from_right(in[0]);
        left = L.begin ? T(0) : left;
        rn = L.end ? T(0) : rn;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const T mid = in[e];
            const T right = seg_right<E>(in, e, rn, L.shortl);
            T k;
            if constexpr (KIND == K_RD) {
                const T loc = fmaT(-mid, fmaT(mid, mid, P.a1), U.at(0, e));
                k = fmaT(left + right, P.a0, loc);
            } else {
                k = fmaT(P.a3, U.at(0, e), fmaT(P.a2, right, fmaT(P.a1, mid, P.a0 * left)));
            }
            left = mid;
            rk_update<STAGE>(k, y[e], acc[e], t[e], st);
        }
    }
}

// Waves per SIMD the registers have to leave room for: y, acc and t are 3 E
// values a lane, per-cell inputs E more.  FP32 instructions of different waves
// overlap, so FP32 gains from a third and fourth wave; FP64 has no use for more
// than two.  What the limit pushes to scratch memory lies in the draws and the
// fold, but for two accesses a step in the FP32 kernels of 48 cells a lane and more
// (480 to 1152 FMAs) and 9 to 32 in the plain FP64 ones of 32 cells with per-cell
// inputs, whose state alone takes 256 registers.
constexpr int mc_min_waves(int size, int E, bool cell_in) {
    const int regs = (cell_in ? 4 : 3) * E * size / 4;
    return regs > 208 ? 1 : size == 8 || regs > 112 ? 2 : regs > 64 ? 3 : 4;
}

template <int KIND, class T, int E, int MODE, bool SEG>
__global__ __launch_bounds__(WAVE * MC_WPB, mc_min_waves(sizeof(T), E, MODE == IN_CELL))
void mc_kernel(McArgs a) {
    using U = typename Key<T>::U;
    __shared__ U kmin[E * WAVE];
    __shared__ U kmax[E * WAVE];
    const int lane = threadIdx.x & (WAVE - 1);
    const int64_t w = (int64_t)blockIdx.x * MC_WPB + threadIdx.x / WAVE;
    const int n = (int)a.n;
    for (int i = threadIdx.x; i < E * WAVE; i += WAVE * MC_WPB) {
        kmin[i] = ~(U)0;
        kmax[i] = 0;
    }
    __syncthreads();

    // this lane's cells: first .. first + cnt - 1 of sample `seg` of a group
    const int L = SEG ? a.L : WAVE;
    const int spw = SEG ? a.spw : 1;
    const int seg = SEG ? lane / L : 0;
    const int ls = lane - seg * L;
    const int F = n - L * (E - 1);
    const Seg S = {SEG && ls >= F, SEG && ls == 0, SEG && ls == L - 1};
    int cnt = SEG ? (S.shortl ? E - 1 : E) : (n - lane * E < 0 ? 0 : n - lane * E > E ? E : n - lane * E);
    if (SEG && seg >= spw) cnt = 0;
    const int first = ls * E - (S.shortl ? ls - F : 0);

    const T* __restrict__ xlo = (const T*)a.x_lo;
    const T* __restrict__ xhi = (const T*)a.x_hi;
    const T* __restrict__ plo = (const T*)a.p_lo;
    const T* __restrict__ phi = (const T*)a.p_hi;
    const SysPrm<T> P = {(T)a.prm[0], (T)a.prm[1], (T)a.prm[2], (T)a.prm[3], (T)a.prm[4]};
    const Steps<T> st = {(T)a.h2, (T)a.dt, (T)a.dt6};
    constexpr bool ZERO = !SEG && E % 4 == 0;

    // waves past nw (in the last workgroup) draw nothing but join the end
    const int64_t groups = w < a.nw ? (a.m + spw - 1) / spw : 0;
    for (int64_t g = w; g < groups; g += a.nw) {
        const int64_t r = g * spw + seg;               // sample of the call
        const bool live = (!SEG || seg < spw) && r < a.m;
        const uint64_t s = (uint64_t)(a.s0 + r);
        T y[1][E];
        Inputs<T, E, 1, MODE> I;
#pragma unroll
        for (int e = 0; e < E; ++e) y[0][e] = ghost<KIND, T>();
        mc_draw<T, E, ZERO>(first, s, a.seed, [&](int e, T u) {
            if (e < cnt) {
                const T lo = xlo[first + e], hi = xhi[first + e];
                y[0][e] = fmaT(u, hi - lo, lo);
            }
        });
        // inputs, drawn per sample at coordinates n + k
        if constexpr (MODE == IN_SCALAR) {
            I.u[0] = T(0);
            if (a.n_in != 0) {
                const U4 b = philox4x64_10((uint64_t)(n >> 2), s, MC_STREAM, 0, a.seed, 0);
                const T u = unif(philox_word(b, n & 3), T(0));
                I.u[0] = fmaT(u, phi[0] - plo[0], plo[0]);
            }
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e) I.u[0][e] = T(0);
            mc_draw<T, E, false>(n + first, s, a.seed, [&](int e, T u) {
                if (e < cnt) {
                    const T lo = plo[first + e], hi = phi[first + e];
                    I.u[0][e] = fmaT(u, hi - lo, lo);
                }
            });
        }

        if constexpr (SEG) {
            T acc[E], t[E];
            const auto step = [&] {
                seg_stage<KIND, 1>(y[0], acc, t, P, I, st, S);
                seg_stage<KIND, 2>(y[0], acc, t, P, I, st, S);
                seg_stage<KIND, 3>(y[0], acc, t, P, I, st, S);
                seg_stage<KIND, 4>(y[0], acc, t, P, I, st, S);
            };
            int64_t k = 0;
            if constexpr (E * sizeof(T) <= 16) {   // (see rk4_steps)
                for (; k + 4 <= a.nsteps; k += 4) {
                    step();
                    step();
                    step();
                    step();
                }
            }
            for (; k < a.nsteps; ++k) step();
        } else if (E * sizeof(T) <= 128 || n == WAVE * E) {   // (see mc_plan)
            Mask<E, false, true> M{E};
            rk4_steps<KIND, T, E, 1, MODE>(y, a.nsteps, P, I, st, M);
        } else {
            Mask<E, true, true> M{cnt};
            rk4_steps<KIND, T, E, 1, MODE>(y, a.nsteps, P, I, st, M);
        }

        // cell j = first + e in slot (j mod E) * 64 + j / E (plain layout: slot
        // e * 64 + lane, no bank conflict)
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if (live && e < cnt) {
                const int j = first + e;
                const int idx = SEG ? (j % E) * WAVE + j / E : e * WAVE + lane;
                const U k = to_key(y[0][e]);
                const bool nan = y[0][e] != y[0][e];
                atomicMin(&kmin[idx], nan ? (U)0 : k);
                atomicMax(&kmax[idx], nan ? ~(U)0 : k);
            }
            if (e % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
    }

    // the group's min / max, cell by cell
    __syncthreads();
    T* __restrict__ pmin = (T*)a.part_min + (size_t)blockIdx.x * n;
    T* __restrict__ pmax = (T*)a.part_max + (size_t)blockIdx.x * n;
    for (int j = threadIdx.x; j < n; j += WAVE * MC_WPB) {
        const int idx = (j % E) * WAVE + j / E;
        pmin[j] = from_key<T>(kmin[idx]);
        pmax[j] = from_key<T>(kmax[idx]);
    }
}

template <int KIND, class T, int E, int MODE, bool SEG>
static hipError_t go(const McArgs& a, hipStream_t s) {
    const unsigned grid = (unsigned)((a.nw + MC_WPB - 1) / MC_WPB);
    hipLaunchKernelGGL((mc_kernel<KIND, T, E, MODE, SEG>), dim3(grid), dim3(WAVE * MC_WPB), 0, s, a);
    return hipGetLastError();
}

// a.L = 0: plain layout.
template <int KIND, class T, int MODE>
static hipError_t by_E(int E, const McArgs& a, hipStream_t s) {
    constexpr bool F32 = sizeof(T) == 4;
    if (a.L == 0) {
        switch (E) {
            case 1: return go<KIND, T, 1, MODE, false>(a, s);
            case 2: return go<KIND, T, 2, MODE, false>(a, s);
            case 4: return go<KIND, T, 4, MODE, false>(a, s);
            case 8: return go<KIND, T, 8, MODE, false>(a, s);
            case 16: return go<KIND, T, 16, MODE, false>(a, s);
            case 32: return go<KIND, T, 32, MODE, false>(a, s);
            case 64: if constexpr (F32) return go<KIND, T, 64, MODE, false>(a, s);
        }
        return hipErrorInvalidValue;
    }
    switch (E) {
        case 1: return go<KIND, T, 1, MODE, true>(a, s);
        case 2: return go<KIND, T, 2, MODE, true>(a, s);
        case 4: return go<KIND, T, 4, MODE, true>(a, s);
        case 6: return go<KIND, T, 6, MODE, true>(a, s);
        case 8: return go<KIND, T, 8, MODE, true>(a, s);
        case 10: return go<KIND, T, 10, MODE, true>(a, s);
        case 12: return go<KIND, T, 12, MODE, true>(a, s);
        case 14: return go<KIND, T, 14, MODE, true>(a, s);
        case 16: return go<KIND, T, 16, MODE, true>(a, s);
        case 18: return go<KIND, T, 18, MODE, true>(a, s);
        case 20: return go<KIND, T, 20, MODE, true>(a, s);
        case 24: return go<KIND, T, 24, MODE, true>(a, s);
        case 28: return go<KIND, T, 28, MODE, true>(a, s);
        case 32: return go<KIND, T, 32, MODE, true>(a, s);
        case 40: if constexpr (F32) return go<KIND, T, 40, MODE, true>(a, s); break;
        case 48: if constexpr (F32) return go<KIND, T, 48, MODE, true>(a, s); break;
        case 56: if constexpr (F32) return go<KIND, T, 56, MODE, true>(a, s); break;
        case 60: if constexpr (F32) return go<KIND, T, 60, MODE, true>(a, s); break;
        case 64: if constexpr (F32) return go<KIND, T, 64, MODE, true>(a, s); break;
    }
    return hipErrorInvalidValue;
}

}  // namespace reach
