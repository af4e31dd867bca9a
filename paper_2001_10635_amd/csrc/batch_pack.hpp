// Device code the batch sources share: the balanced layout of a query over
// lanes, its RK4 stages, and segment packs (see batch.hip).
#pragma once
#include "dev.hpp"
#include "kernels.hpp"

namespace reach {

__device__ __forceinline__ uint64_t wave_bcast(uint64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// Balanced layout of a query's n cells over the 64 lanes: E = ceil(n / 64)
// (1..8), the first F = n - 64 (E - 1) lanes hold E consecutive cells and the
// others ("short" lanes) E - 1.  For E >= 2 every lane holds cells and the
// chain's last cell sits in lane 63, so no cell of the window is a ghost and
// no stage needs a per-cell select: a short lane's last cell is slot E - 2,
// whose right neighbour (and the value its left neighbour lane reads) is
// picked once per stage; slot E - 1 of a short lane computes a value nobody
// reads.  For E = 1 the lanes past cell n-1 are empty and the right neighbour
// of cell n-1 is set to the ghost.  The arithmetic per cell is the
// large-chain kernel's, operation for operation, so a query's box is the
// same alone, batched or served.
struct Lanes {
    bool shortl;   // this lane holds E - 1 cells
    bool begin;    // this lane holds cell 0 (read by segment packs only)
    bool end;      // this lane holds cell n-1
    int cnt;       // cells held
    int64_t first; // index of the first cell held
};

template <int E>
__device__ __forceinline__ Lanes lanes_of(int64_t n) {
    const int lane = threadIdx.x;
    const int64_t F = n - (int64_t)WAVE * (E - 1);   // lanes holding E cells
    Lanes L;
    L.shortl = lane >= F;
    L.cnt = L.shortl ? E - 1 : E;
    L.first = (int64_t)lane * E - (L.shortl ? (int64_t)lane - F : 0);
    L.begin = lane == 0;
    L.end = (E == 1) ? (lane == n - 1) : (lane == WAVE - 1);
    return L;
}

// Right neighbour of slot e, given the value shifted in from the next lane.
template <int E, class T>
__device__ __forceinline__ T right_of(const T (&in)[E], int e, T rn, bool shortl) {
    if (e == E - 1) return rn;
    if (e == E - 2) return shortl ? rn : in[E - 1];
    return in[e + 1];
}
// The value lane l + 1 needs from this lane: its last held cell.
template <int E, class T>
__device__ __forceinline__ T last_of(const T (&in)[E], bool shortl) {
    if constexpr (E == 1) return in[0];
    else return shortl ? in[E - 2] : in[E - 1];
}

// SEG: the query occupies a run of lanes inside the wave (a segment pack), so
// its first lane takes the left boundary value and its last lane the right
// ghost by a select, where a query spanning the whole wave gets them from the
// shifts' zero fill.
template <int KIND, int STAGE, int E, int S, bool SEG = false>
__device__ __forceinline__ void bal_stage(double (&y)[S][E], double (&acc)[S][E],
                                          double (&t)[S][E], const SysPrm<double>& P,
                                          const Inputs<double, E, S, IN_SCALAR>& U,
                                          const Steps<double>& st, const Lanes& L) {
    using T = double;
    T (&in)[S][E] = (STAGE == 1) ? y : t;
    if constexpr (KIND == K_CTM) {
        // F_e = min(v y_e, wc - w y_{e+1}, q), k_e = F_{e-1} - F_e; ghost -inf
        // right of cell n-1 (free outflow), zero flux into cell 0 (lane 0
        // receives 0 from the shift)
        const T v = P.a0, w = P.a1, wc = P.a2, q = P.a3;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            T rn = from_right(in[s][0]);
            rn = L.end ? neg_inf<T>() : rn;
            T F[E];
#pragma unroll
            for (int e = 0; e < E; ++e)
                F[e] = minT(minT(v * in[s][e], fmaT(-w, right_of<E>(in[s], e, rn, L.shortl), wc)), q);
            T Fprev = from_left(last_of<E>(F, L.shortl));
            if (SEG) Fprev = L.begin ? T(0) : Fprev;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const T k = Fprev - F[e];
                Fprev = F[e];
                rk_update<STAGE>(k, y[s][e], acc[s][e], t[s][e], st);
            }
        }
    } else if constexpr (KIND == K_RD) {
        // k = (y_{e-1} + y_{e+1}) / h^2 + (u - y_e (y_e^2 + 2 / h^2)), ghosts 0
        const T ih2 = P.a0, two_ih2 = P.a1;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            T ln = from_left(last_of<E>(in[s], L.shortl));
            if (SEG) ln = L.begin ? T(0) : ln;
            T rn = from_right(in[s][0]);
            if (E == 1 || SEG) rn = L.end ? T(0) : rn;
            T left = ln;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const T mid = in[s][e];
                const T right = right_of<E>(in[s], e, rn, L.shortl);
                const T loc = fmaT(-mid, fmaT(mid, mid, two_ih2), U.at(s, e));
                const T k = fmaT(left + right, ih2, loc);
                left = mid;
                rk_update<STAGE>(k, y[s][e], acc[s][e], t[s][e], st);
            }
        }
    } else {
        // LIN3, both sides (S == 2): the sign split of aL, aR, b
        const T aL = P.a0, aD = P.a1, aR = P.a2, b = P.a3;
        const T aLp = aL > T(0) ? aL : T(0), aLn = aL < T(0) ? aL : T(0);
        const T aRp = aR > T(0) ? aR : T(0), aRn = aR < T(0) ? aR : T(0);
        const T bp = b > T(0) ? b : T(0), bn = b < T(0) ? b : T(0);
        T ln[2], rn[2], left[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            ln[s] = from_left(last_of<E>(in[s], L.shortl));
            if (SEG) ln[s] = L.begin ? T(0) : ln[s];
            rn[s] = from_right(in[s][0]);
            if (E == 1 || SEG) rn[s] = L.end ? T(0) : rn[s];
            left[s] = ln[s];
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            T mid[2], right[2], k[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                mid[s] = in[s][e];
                right[s] = right_of<E>(in[s], e, rn[s], L.shortl);
            }
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int o = 1 - s;
                T acc0 = aD * mid[s];
                acc0 = fmaT(aLp, left[s], acc0);
                acc0 = fmaT(aLn, left[o], acc0);
                acc0 = fmaT(aRp, right[s], acc0);
                acc0 = fmaT(aRn, right[o], acc0);
                acc0 = fmaT(bp, U.at(s, e), acc0);
                k[s] = fmaT(bn, U.at(o, e), acc0);
            }
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                left[s] = mid[s];
                rk_update<STAGE>(k[s], y[s][e], acc[s][e], t[s][e], st);
            }
        }
    }
}

// Segment packs: several queries of one kind with bitwise equal constants and
// dt share a wave, E cells per lane (E = 2, 4, 8 or 16, one E per pack).  Member m
// runs on the L_m = ceil(n_m / E) lanes after the previous members', in the
// balanced layout of those lanes: the first F_m = n_m - L_m (E - 1) lanes hold
// E cells and the others E - 1 (the planner packs a query at this E only when
// F_m >= 0).  A member's first and last lanes take the chain's boundary values
// by a select, so members never read each other's cells; lanes past the last
// member hold ghosts and stay masked off.  The wave runs the longest member's
// steps, a member's lanes masked off once its own steps are done.  Per cell
// this is the single-query arithmetic, so every box is bitwise the one the
// query gets alone.
//
// S = 1 runs only side `side` of a pack of a cooperative system: the longest
// packs of a batch go to two waves, one per side, where a single wave would hold
// up the end of the launch (see plan_batch); `pair` counts the pack's finished
// sides, and the wave that finishes last checks the order.
template <int KIND, int E, int S>
__device__ __forceinline__ void run_seg(const QDesc* __restrict__ desc,
                                     const uint32_t* __restrict__ mem_idx, int count, int side,
                                     unsigned int* pair, unsigned int* qflags,
                                     unsigned int* status) {
    using T = double;
    const int lane = threadIdx.x;
    const QDesc* d0 = desc + mem_idx[0];
    int mem = -1, off = 0, base = 0, len = 0;
    int64_t steps = 0;   // the longest member's
    for (int m = 0; m < count; ++m) {
        const QDesc* dm = desc + mem_idx[m];
        const int l = (int)((dm->n + E - 1) / E);
        if (lane >= off && lane < off + l) {
            mem = m;
            base = off;
            len = l;
        }
        off += l;
        steps = dm->nsteps > steps ? dm->nsteps : steps;
    }
    const bool valid = mem >= 0;
    const QDesc* me = desc + mem_idx[valid ? mem : 0];
    const int64_t n = me->n;
    const int rel = lane - base;
    const int64_t F = n - (int64_t)len * (E - 1);   // lanes holding E cells
    Lanes L;
    L.shortl = rel >= F;
    L.cnt = !valid ? 0 : (L.shortl ? E - 1 : E);
    L.first = (int64_t)rel * E - (L.shortl ? (int64_t)rel - F : 0);
    L.begin = valid && rel == 0;
    L.end = valid && rel == len - 1;
    const double* src[2] = {me->x_lo, me->x_hi};
    const double* pin[2] = {me->p_lo, me->p_hi};
    T y[S][E];
    Inputs<T, E, S, IN_SCALAR> U;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const int sd = S == 1 ? side : s;
#pragma unroll
        for (int e = 0; e < E; ++e)
            y[s][e] = (e < L.cnt) ? src[sd][L.first + e] : ghost<KIND, T>();
        U.u[s] = (valid && pin[sd]) ? *pin[sd] : T(0);
    }
    SysPrm<T> P;
    P.a0 = d0->prm[0]; P.a1 = d0->prm[1]; P.a2 = d0->prm[2]; P.a3 = d0->prm[3]; P.a4 = d0->prm[4];
    const Steps<T> st = {d0->h2, d0->dt, d0->dt6};
    T acc[S][E], t[S][E];
    const int64_t mine = valid ? me->nsteps : 0;
    for (int64_t k = 0; k < steps; ++k) {
        if (k < mine) {
            bal_stage<KIND, 1, E, S, true>(y, acc, t, P, U, st, L);
            bal_stage<KIND, 2, E, S, true>(y, acc, t, P, U, st, L);
            bal_stage<KIND, 3, E, S, true>(y, acc, t, P, U, st, L);
            bal_stage<KIND, 4, E, S, true>(y, acc, t, P, U, st, L);
        }
    }
    unsigned bits = 0;
    double* dst[2] = {me->r_lo, me->r_hi};
#pragma unroll
    for (int e = 0; e < E; ++e) {
        if (e < L.cnt) {
            const int64_t j = L.first + e;
#pragma unroll
            for (int s = 0; s < S; ++s) {
                dst[S == 1 ? side : s][j] = y[s][e];
                if (!finiteT(y[s][e])) bits |= ST_NONFINITE;
            }
            if constexpr (S == 2) {
                if (y[0][e] > y[1][e]) bits |= ST_ORDER;
            }
        }
    }
    if constexpr (S == 1) {
        // publish this side, then the second side to finish checks the order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        uint64_t old = 0;
        if (lane == 0)
            old = __hip_atomic_fetch_add(pair, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        if (wave_bcast(old) == 1) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
#pragma unroll
            for (int e = 0; e < E; ++e) {
                if (e < L.cnt) {
                    const T o = dst[1 - side][L.first + e];
                    if (side == 0 ? y[0][e] > o : o > y[0][e]) bits |= ST_ORDER;
                }
            }
        }
    }
    if (bits) {
        atomicOr(&qflags[me->tag], bits);
        atomicOr(status, bits);
    }
}

// Persistent worker of a packed batch: every item is a segment pack.  The
// packs' bodies are inlined into this one kernel (no calls).  EMAX is the
// widest pack it runs: with EMAX = 8 its registers are capped for three waves
// per SIMD (it runs fastest at two); the 16-cell bodies need ~240 registers,
// so EMAX = 16 fits two waves per SIMD and runs fastest at one, whose 32
// independent cell-sides per stage keep the SIMD issuing.
// n_items: the item count in its low half; the first (its high half) of them
// run one side per wave (SIDES).
template <int EMAX, bool SIDES>
__device__ __forceinline__ void pack_items(
        const QDesc* __restrict__ desc, const BatchItem* __restrict__ items,
        const uint32_t* __restrict__ members, const uint64_t* n_items,
        unsigned long long* counter, unsigned int* qflags, unsigned int* pair,
        unsigned int* status) {
    const int lane = threadIdx.x;
    const uint64_t nw = wave_bcast(*n_items);
    const uint64_t ni = SIDES ? nw & 0xFFFFFFFFu : nw, ns = SIDES ? nw >> 32 : 0;
    for (;;) {
        uint64_t u = 0;
        if (lane == 0) u = atomicAdd(counter, 1ULL);
        u = wave_bcast(u);
        if (u >= ni + ns) break;
        const bool one = SIDES && u < 2 * ns;        // one side of item u / 2
        const uint64_t i = one ? u >> 1 : u - ns;
        const int side = SIDES ? (int)(u & 1) : 0;
        const BatchItem it = items[i];
        const int kind = desc[members[it.start]].kind;
        const uint32_t* mi = members + it.start;
        const int cnt = it.count;
        const int ki = kind == K_CTM ? 0 : kind == K_RD ? 1 : 2;
        const int ei = it.E == 2 ? 0 : it.E == 4 ? 1 : it.E == 8 ? 2 : 3;
#define REACH_PACK(KIND, E, S) run_seg<KIND, E, S>(desc, mi, cnt, side, pair + i, qflags, status)
        if constexpr (SIDES) {
            if (one && ki < 2) {
                switch (4 * ki + ei) {
                    case 0: REACH_PACK(K_CTM, 2, 1); break;
                    case 1: REACH_PACK(K_CTM, 4, 1); break;
                    case 2: REACH_PACK(K_CTM, 8, 1); break;
                    case 4: REACH_PACK(K_RD, 2, 1); break;
                    case 5: REACH_PACK(K_RD, 4, 1); break;
                    case 6: REACH_PACK(K_RD, 8, 1); break;
                    default:
                        if constexpr (EMAX > 8) {
                            if (ki == 0) REACH_PACK(K_CTM, 16, 1);
                            else REACH_PACK(K_RD, 16, 1);
                        }
                        break;
                }
                continue;
            }
            if (one && side == 1) continue;              // a coupled pack ran whole as side 0
        }
        switch (4 * ki + ei) {
            case 0: REACH_PACK(K_CTM, 2, 2); break;
            case 1: REACH_PACK(K_CTM, 4, 2); break;
            case 2: REACH_PACK(K_CTM, 8, 2); break;
            case 4: REACH_PACK(K_RD, 2, 2); break;
            case 5: REACH_PACK(K_RD, 4, 2); break;
            case 6: REACH_PACK(K_RD, 8, 2); break;
            case 8: REACH_PACK(K_LIN3, 2, 2); break;
            case 9: REACH_PACK(K_LIN3, 4, 2); break;
            case 10: REACH_PACK(K_LIN3, 8, 2); break;
            default:   // E = 16 (the host gives such packs to EMAX = 16 only)
                if constexpr (EMAX > 8) {
                    if (ki == 0) REACH_PACK(K_CTM, 16, 2);
                    else if (ki == 1) REACH_PACK(K_RD, 16, 2);
                    else REACH_PACK(K_LIN3, 16, 2);
                }
                break;
        }
#undef REACH_PACK
    }
}

template <int EMAX>
__global__ __launch_bounds__(64, EMAX > 8 ? 2 : 3) void pack_kernel(
        const QDesc* __restrict__ desc, const BatchItem* __restrict__ items,
        const uint32_t* __restrict__ members, const uint64_t* n_items,
        unsigned long long* counter, unsigned int* qflags, unsigned int* status) {
    pack_items<EMAX, false>(desc, items, members, n_items, counter, qflags, nullptr, status);
}

template <int EMAX>
__global__ __launch_bounds__(64, EMAX > 8 ? 2 : 3) void pack_sides_kernel(
        const QDesc* __restrict__ desc, const BatchItem* __restrict__ items,
        const uint32_t* __restrict__ members, const uint64_t* n_items,
        unsigned long long* counter, unsigned int* qflags, unsigned int* pair,
        unsigned int* status) {
    pack_items<EMAX, true>(desc, items, members, n_items, counter, qflags, pair, status);
}

}  // namespace reach
