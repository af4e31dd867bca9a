// Device building blocks for the gfx950 reachability kernels.
//
// Layout convention shared by every kernel: one wavefront (64 lanes) owns a
// window of 64*E consecutive cells of a chain, lane l holding cells
// [l*E, l*E + E) of the window in registers.  A three-point stencil then
// needs only two cross-lane values per stage (the last cell of lane l-1 and
// the first cell of lane l+1), moved with DPP whole-wave shifts; every other
// neighbour is a register of the same lane.  Lanes past either end of the
// wave receive zero, which is how the chain's boundary conditions enter when
// the window starts at cell 0 or ends at cell n-1 (see Mask below).
//
// The four stages of classical RK4 (Algorithm 1, read as the classical
// method: stage inputs z + dt/2 K1, z + dt/2 K2, z + dt K3, update
// z + dt/6 (K1 + 2 K2 + 2 K3 + K4)) run on registers: per cell and side the
// state y, the running sum acc = K1 + 2 K2 + 2 K3 + K4 and the current stage
// input t.  No stage value ever leaves the register file.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace reach {

constexpr int WAVE = 64;

// DPP controls of the GFX9 family: shift the whole wavefront by one lane.
constexpr int DPP_WAVE_SHL1 = 0x130;  // lane l reads lane l+1
constexpr int DPP_WAVE_SHR1 = 0x138;  // lane l reads lane l-1

// Lane l receives x of lane l-1; lane 0 receives 0 (DPP bound control: the
// out-of-wave source reads as zero, so no fill value has to be staged).
__device__ __forceinline__ float from_left(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), DPP_WAVE_SHR1, 0xF,
                                                      0xF, true));
}
// Lane l receives x of lane l+1; lane 63 receives 0.
__device__ __forceinline__ float from_right(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), DPP_WAVE_SHL1, 0xF,
                                                      0xF, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp64(double x) {
    const uint64_t xi = (uint64_t)__double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)xi, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(xi >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}
__device__ __forceinline__ double from_left(double x) { return dpp64<DPP_WAVE_SHR1>(x); }
__device__ __forceinline__ double from_right(double x) { return dpp64<DPP_WAVE_SHL1>(x); }

// Lane l receives x of lane l+1; lane 63 keeps `last` (a shift without a source
// lane leaves its destination unwritten), so no select follows the shift.
__device__ __forceinline__ float from_right_or(float x, float last) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(last), __float_as_int(x),
                                                      DPP_WAVE_SHL1, 0xF, 0xF, false));
}
__device__ __forceinline__ double from_right_or(double x, double last) {
    const uint64_t xi = (uint64_t)__double_as_longlong(x);
    const uint64_t li = (uint64_t)__double_as_longlong(last);
    const int lo = __builtin_amdgcn_update_dpp((int)(uint32_t)li, (int)(uint32_t)xi, DPP_WAVE_SHL1,
                                               0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(uint32_t)(li >> 32), (int)(uint32_t)(xi >> 32),
                                               DPP_WAVE_SHL1, 0xF, 0xF, false);
    return __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}

__device__ __forceinline__ float fmaT(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmaT(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float minT(float a, float b) { return __builtin_fminf(a, b); }
__device__ __forceinline__ double minT(double a, double b) { return __builtin_fmin(a, b); }

// min with an operand that came through a lane shift: the compiler cannot see
// that the value is no signalling NaN and would put a max(x, x) before the min
// (in the dependent chain of every stage).
__device__ __forceinline__ float min_shifted(float a, float b) {
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ double min_shifted(double a, double b) {
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

template <class T> __device__ __forceinline__ T neg_inf();
template <> __device__ __forceinline__ float neg_inf<float>() { return -__builtin_inff(); }
template <> __device__ __forceinline__ double neg_inf<double>() { return -__builtin_inf(); }

// ------------------------------------------------------------- systems --
// Kind tags (match the C ABI) and input modes.  K_LIN3C and K_LIN3M are the
// LIN3 embedding with the signs of its couplings known (both sides per wave):
//   C  neither neighbour's term crosses to the other side,
//   M  the left neighbour's does, the right one's does not.
// The other sign patterns become these two by exchanging the sides of every
// odd cell (see embed_tile_kernel).
enum { K_CTM = 1, K_RD = 2, K_LIN3 = 3, K_LIN3C = 13, K_LIN3M = 14 };
enum { IN_SCALAR = 0, IN_CELL = 1, IN_ALT = 2 };

// Per-launch system constants, already converted to the kernel's type.
template <class T> struct SysPrm {
    T a0, a1, a2, a3, a4;   // CTM: v, w, c*w, q  RD: 1/h^2, 2/h^2  LIN3: aL, aD, aR, b
};

// Inputs seen by one lane: scalar (same for every cell), one per cell, or one
// for the even and one for the odd slots (IN_ALT: a scalar input in a LIN3
// wave, which may exchange the sides of its odd cells).
template <class T, int E, int S, int MODE> struct Inputs;
template <class T, int E, int S> struct Inputs<T, E, S, IN_SCALAR> {
    T u[S];
    __device__ __forceinline__ T at(int s, int) const { return u[s]; }
};
template <class T, int E, int S> struct Inputs<T, E, S, IN_CELL> {
    T u[S][E];
    __device__ __forceinline__ T at(int s, int e) const { return u[s][e]; }
};
template <class T, int E, int S> struct Inputs<T, E, S, IN_ALT> {
    T u[S][2];
    __device__ __forceinline__ T at(int s, int e) const { return u[s][e & 1]; }
};

// Stage update applied to cell e of side s once its derivative k is known.
// STAGE 1..4 of classical RK4; h2 = dt/2, dt, dt6 = dt/6.
template <class T> struct Steps { T h2, dt, dt6; };

template <int STAGE, class T>
__device__ __forceinline__ void rk_update(T k, T& y, T& acc, T& t, const Steps<T>& st) {
    if (STAGE == 1) { acc = k;                 t = fmaT(st.h2, k, y); }
    if (STAGE == 2) { acc = fmaT(T(2), k, acc); t = fmaT(st.h2, k, y); }
    if (STAGE == 3) { acc = fmaT(T(2), k, acc); t = fmaT(st.dt, k, y); }
    if (STAGE == 4) { acc = acc + k;           y = fmaT(st.dt6, acc, y); }
}

// Where a window sits relative to the chain's right end.
//   PAD : the window runs past cell n-1; cells at or beyond n hold the
//         boundary's ghost value at every stage (nvalid cells of this lane are
//         inside the chain): a select per cell.
//   ONE : (with PAD; waves that hold one side) only cell n, the right
//         neighbour of cell n-1, is set to the ghost after each stage: slot `en` of the lane holding it, en the same in every
//         lane, so one indexed register move per stage replaces the per-cell
//         selects.  Cells beyond n then hold values that reach no cell of the
//         chain and that no caller reads or checks.  Only for lane arrays of
//         up to 128 bytes: an index into longer ones (or into both sides of a
//         window) made the compiler move them to scratch memory.
//   END : the window contains cell n-1, so lane 63's right neighbour is the
//         ghost.  Zero-filled lane shifts already give the Dirichlet ghost 0;
//         only the CTM's free outflow (ghost -inf) needs an explicit value.
// A window's left end at cell 0 needs nothing: lane 0 receives 0 from the
// left, which is both the Dirichlet ghost and the CTM's zero inflow flux.
template <int E, bool PAD, bool END, bool ONE = false> struct Mask {
    int nvalid;  // cells of this lane inside the chain
    int en;      // slot of cell n in its lane (wave-uniform; ONE only)
    bool mine;   // this lane holds cell n (ONE only)
    template <class T> static constexpr bool indexed() { return PAD && ONE && E * sizeof(T) <= 128; }
    template <class T> static constexpr bool per_cell() { return PAD && !indexed<T>(); }
    __device__ __forceinline__ bool ok(int e) const { return !PAD || e < nvalid; }
    template <class T>
    __device__ __forceinline__ void fix(T (&v)[E], T ghost) const {
        if constexpr (indexed<T>()) {
            const T cur = v[en];
            v[en] = mine ? ghost : cur;
        }
    }
};

// The mask of a window whose first n_rel cells (1 <= n_rel <= 64 E) are the
// chain's (cell n is the window's cell n_rel).
template <int E, bool END, bool ONE = false>
__device__ __forceinline__ Mask<E, true, END, ONE> chain_end_mask(int64_t n_rel) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int64_t left = n_rel - (int64_t)lane * E;
    Mask<E, true, END, ONE> M;
    M.nvalid = (int)(left < 0 ? 0 : (left > E ? E : left));
    M.en = 0;
    M.mine = false;
    if constexpr (ONE) {
        M.en = __builtin_amdgcn_readfirstlane((int)(n_rel % E));
        M.mine = lane == (int)(n_rel / E);
    }
    return M;
}

// Ghost value of a system past the chain's right end.
template <int KIND, class T> __device__ __forceinline__ T ghost() {
    if constexpr (KIND == K_CTM) return neg_inf<T>();
    else return T(0);
}

// What a lane holds of its neighbour lanes' edge cells, for the stage input at
// hand: r, the first cell of lane l+1, and l, the last cell of lane l-1.  For the
// CTM r is the supply w (c - y) of that cell, and l is not used: the left lane
// hands over its outgoing flux.
template <class T, int S> struct Edges {
    T l[S], r[S];
};

// Whether a stage hands its edge cells on as soon as they are known: not in the
// widest windows, where the values held meanwhile cost registers and the inner
// cells cover the shifts anyway, nor at two RD cells, which are both edges (5%
// slower there; the CTM's fluxes between them leave work to overlap).
template <int KIND, class T, int E> constexpr bool early_edges() {
    return E * sizeof(T) <= 128 && !(KIND == K_RD && E == 2);
}

template <int KIND, class T, int E, int S, bool END>
__device__ __forceinline__ void get_edges(Edges<T, S>& c, const T (&in)[E], int s,
                                          const SysPrm<T>& P) {
    if constexpr (KIND == K_CTM) {
        // END: lane 63 keeps the ghost's supply from first_edges
        const T sup = fmaT(-P.a1, in[0], P.a2);
        c.r[s] = END ? from_right_or(sup, c.r[s]) : from_right(sup);
    } else {
        c.l[s] = from_left(in[E - 1]);
        c.r[s] = from_right(in[0]);
    }
}

// Before the first get_edges.
template <int KIND, class T, int S>
__device__ __forceinline__ void first_edges(Edges<T, S>& c, const SysPrm<T>& P) {
    if constexpr (KIND == K_CTM) {
#pragma unroll
        for (int s = 0; s < S; ++s) c.r[s] = fmaT(-P.a1, neg_inf<T>(), P.a2);
    }
}

// One RK4 stage for all cells of the lane, for every side s < S.
//   in  : the stage input (y for stage 1, t otherwise)
//   c   : the neighbour lanes' edge cells of `in`; on return those of the next
//         stage's input (early_edges; else read here)
// For S == 2 the sides are (lower, upper) of the embedding; for S == 1 the
// kernel integrates f itself (Monte Carlo) or one side of a cooperative chain.
//
// The lane's two edge cells are computed first and (early_edges) handed to the
// neighbour lanes at once, so that the lane shifts (two moves of a double, each
// waiting for the cell's update) run while the inner cells are computed instead
// of holding up the next stage.  A wave alone on its SIMD, as on every chain too
// short to fill the chip, has nothing else to issue meanwhile (RD FP64, 4 cells
// a lane: 0.30 -> 0.25 us a step).
template <int KIND, int STAGE, class T, int E, int S, int MODE, bool MASKED, bool END, bool ONE>
__device__ __forceinline__ void rk_stage(T (&y)[S][E], T (&acc)[S][E], T (&t)[S][E],
                                         const SysPrm<T>& P, const Inputs<T, E, S, MODE>& U,
                                         const Steps<T>& st, const Mask<E, MASKED, END, ONE>& M,
                                         Edges<T, S>& c)
{
    T (&in)[S][E] = (STAGE == 1) ? y : t;
    T (&out)[S][E] = (STAGE == 4) ? y : t;
    constexpr bool FIX = Mask<E, MASKED, END, ONE>::template indexed<T>();
    constexpr bool EARLY = !FIX && early_edges<KIND, T, E>();
    if constexpr (!EARLY) {
#pragma unroll
        for (int s = 0; s < S; ++s) get_edges<KIND, T, E, S, END>(c, in[s], s, P);
    }
    const auto put = [&](int s, int e, T k) {
        rk_update<STAGE>(k, y[s][e], acc[s][e], t[s][e], st);
        if (M.template per_cell<T>() && !M.ok(e)) out[s][e] = ghost<KIND, T>();
    };
    // the ghost's slot (a padded window)
    const auto finish = [&](int s) {
        if constexpr (FIX) M.fix(out[s], ghost<KIND, T>());
    };
    if constexpr (KIND == K_CTM) {
        // Flux form: F_e = min(v y_e, w (c - y_{e+1}), q) = min(demand of e,
        // supply of e+1) with demand min(v y, q) and supply wc - w y,
        // k_e = F_{e-1} - F_e.  Right ghost past the chain's end is -inf, so
        // its supply is +inf (free outflow); the flux into the window's first
        // cell arrives from the left lane, 0 at lane 0 (zero inflow into cell 0).
        const T v = P.a0, w = P.a1, wc = P.a2, q = P.a3;
        const auto flux = [&](T ye, T yr) { return minT(minT(v * ye, q), fmaT(-w, yr, wc)); };
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const T o0 = in[s][0], oE = in[s][E - 1];
            const T Fout = min_shifted(minT(v * oE, q), c.r[s]);
            const T Fin = from_left(Fout);
            const T F0 = E > 1 ? flux(o0, in[s][1]) : Fout;
            T Fprev = F0;
            const T FE = E > 2 ? flux(in[s][E - 2], oE) : F0;   // into the last cell
            if constexpr (E > 1) put(s, E - 1, FE - Fout);
            put(s, 0, Fin - F0);
            if constexpr (EARLY) get_edges<KIND, T, E, S, END>(c, out[s], s, P);
#pragma unroll
            for (int e = 1; e < E - 1; ++e) {
                const T F = (e == E - 2) ? FE : flux(in[s][e], in[s][e + 1]);
                const T k = Fprev - F;
                Fprev = F;
                put(s, e, k);
            }
            finish(s);
        }
    } else if constexpr (KIND == K_RD || S == 1) {
        const auto f = [&](int s, int e, T left, T mid, T right) {
            if constexpr (KIND == K_RD) {
                // k = (y_{e-1} - 2 y_e + y_{e+1}) / h^2 - y_e^3 + u, Dirichlet
                // ghosts 0, regrouped into four fused operations:
                //   k = (y_{e-1} + y_{e+1}) / h^2 + (u - y_e (y_e^2 + 2 / h^2)).
                const T loc = fmaT(-mid, fmaT(mid, mid, P.a1), U.at(s, e));
                return fmaT(left + right, P.a0, loc);
            } else {
                // LIN3, f = aL y_{e-1} + aD y_e + aR y_{e+1} + b u
                return fmaT(P.a3, U.at(s, e), fmaT(P.a2, right, fmaT(P.a1, mid, P.a0 * left)));
            }
        };
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if constexpr (!EARLY) {
                T left = c.l[s];
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const T mid = in[s][e];
                    const T k = f(s, e, left, mid, (e == E - 1) ? c.r[s] : in[s][e + 1]);
                    left = mid;
                    put(s, e, k);
                }
                finish(s);
                continue;
            }
            const T o0 = in[s][0], oE = in[s][E - 1];
            if constexpr (E == 1) {
                put(s, 0, f(s, 0, c.l[s], o0, c.r[s]));
            } else {
                const T k0 = f(s, 0, c.l[s], o0, in[s][1]);
                const T kE = f(s, E - 1, in[s][E - 2], oE, c.r[s]);
                put(s, 0, k0);
                put(s, E - 1, kE);
            }
            if constexpr (EARLY) get_edges<KIND, T, E, S, END>(c, out[s], s, P);
            T left = o0;
#pragma unroll
            for (int e = 1; e < E - 1; ++e) {
                const T mid = in[s][e];
                const T k = f(s, e, left, mid, (e == E - 2) ? oE : in[s][e + 1]);
                left = mid;
                put(s, e, k);
            }
            finish(s);
        }
    } else {
        // LIN3 embedding, d(x, p, xh, ph) with the sign split of aL, aR, b; both
        // sides of a cell are computed from the old values before either is
        // updated.
        static_assert(S == 2, "the coupled chain holds both sides");
        const T aL = P.a0, aD = P.a1, aR = P.a2, b = P.a3;
        const auto d = [&](int s, int e, const T (&left)[2], const T (&mid)[2],
                           const T (&right)[2]) {
            const int o = 1 - s;
            T k = aD * mid[s];
            if constexpr (KIND == K_LIN3) {
                const T aLp = aL > T(0) ? aL : T(0), aLn = aL < T(0) ? aL : T(0);
                const T aRp = aR > T(0) ? aR : T(0), aRn = aR < T(0) ? aR : T(0);
                const T bp = b > T(0) ? b : T(0), bn = b < T(0) ? b : T(0);
                k = fmaT(aLp, left[s], k);
                k = fmaT(aLn, left[o], k);
                k = fmaT(aRp, right[s], k);
                k = fmaT(aRn, right[o], k);
                k = fmaT(bp, U.at(s, e), k);
                return fmaT(bn, U.at(o, e), k);
            } else {
                // the terms with a nonzero coefficient, in the same order; U
                // holds the input of the side that b selects
                k = fmaT(aL, left[KIND == K_LIN3M ? o : s], k);
                k = fmaT(aR, right[s], k);
                return fmaT(b, U.at(s, e), k);
            }
        };
        T o0[2], oE[2], k0[2], kE[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            o0[s] = in[s][0];
            oE[s] = in[s][E - 1];
        }
        if constexpr (E == 1) {
#pragma unroll
            for (int s = 0; s < 2; ++s) k0[s] = d(s, 0, c.l, o0, c.r);
        } else {
            const T i1[2] = {in[0][1], in[1][1]}, iE[2] = {in[0][E - 2], in[1][E - 2]};
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                k0[s] = d(s, 0, c.l, o0, i1);
                kE[s] = d(s, E - 1, iE, oE, c.r);
            }
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            put(s, 0, k0[s]);
            if constexpr (E > 1) put(s, E - 1, kE[s]);
        }
#pragma unroll
        for (int s = 0; s < 2; ++s)
            if constexpr (EARLY) get_edges<KIND, T, E, S, END>(c, out[s], s, P);
        T left[2] = {o0[0], o0[1]};
#pragma unroll
        for (int e = 1; e < E - 1; ++e) {
            const T mid[2] = {in[0][e], in[1][e]};
            T right[2], k[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) right[s] = (e == E - 2) ? oE[s] : in[s][e + 1];
#pragma unroll
            for (int s = 0; s < 2; ++s) k[s] = d(s, e, left, mid, right);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                left[s] = mid[s];
                put(s, e, k[s]);
            }
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) finish(s);
    }
}

// `nsteps` classical RK4 steps on the lane's registers.
template <int KIND, class T, int E, int S, int MODE, bool MASKED, bool END, bool ONE>
__device__ __forceinline__ void rk4_steps(T (&y)[S][E], int64_t nsteps, const SysPrm<T>& P,
                                          const Inputs<T, E, S, MODE>& U, const Steps<T>& st,
                                          const Mask<E, MASKED, END, ONE>& M)
{
    T acc[S][E], t[S][E];
    Edges<T, S> c;
    first_edges<KIND>(c, P);
    if constexpr (early_edges<KIND, T, E>()) {
#pragma unroll
        for (int s = 0; s < S; ++s) get_edges<KIND, T, E, S, END>(c, y[s], s, P);
    }
    const auto step = [&] {
        rk_stage<KIND, 1>(y, acc, t, P, U, st, M, c);
        rk_stage<KIND, 2>(y, acc, t, P, U, st, M, c);
        rk_stage<KIND, 3>(y, acc, t, P, U, st, M, c);
        rk_stage<KIND, 4>(y, acc, t, P, U, st, M, c);
    };
    // A step of one or two cells is some 45 to 70 instructions, of which the loop's
    // counter, compare and branch would be a tenth: four steps to an iteration
    // (CTM FP64 n = 64, 400 steps: 43.8 us at one step, 38.4 at four), and two for
    // four CTM cells (n = 50000 160 -> 154 us; the RD chain is 3% slower so).
    int64_t k = 0;
    if constexpr (S * E * sizeof(T) <= 16) {
        for (; k + 4 <= nsteps; k += 4) {
            step();
            step();
            step();
            step();
        }
    } else if constexpr (KIND == K_CTM && S * E * sizeof(T) <= 32) {
        for (; k + 2 <= nsteps; k += 2) {
            step();
            step();
        }
    }
    for (; k < nsteps; ++k) step();
}

// ------------------------------------------------------------ status --
// Bits OR-ed into the context's device status word (ST_CANCELLED: only in a
// served query's own flags, never in the context's word).
enum { ST_NONFINITE = 1, ST_ORDER = 2, ST_CANCELLED = 4 };

__device__ __forceinline__ bool finiteT(float x) { return __builtin_isfinite(x); }
__device__ __forceinline__ bool finiteT(double x) { return __builtin_isfinite(x); }

// One lane per wave ORs `bits` (wave-reduced) into *status with a vector atomic.
__device__ __forceinline__ void report_status(unsigned int* status, unsigned int bits) {
    const unsigned long long nf = __ballot(bits & ST_NONFINITE);
    const unsigned long long od = __ballot(bits & ST_ORDER);
    if ((nf | od) && (threadIdx.x & 63) == 0)
        atomicOr(status, (nf ? (unsigned)ST_NONFINITE : 0u) | (od ? (unsigned)ST_ORDER : 0u));
}

// ------------------------------------------------------------ Philox --
// Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC'11): 10 rounds of two
// 64x64->128 multiplications with the published multipliers and Weyl key
// increments.  Used for the Monte Carlo samples.
struct U4 { uint64_t x[4]; };

__device__ __forceinline__ U4 philox4x64_10(uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3,
                                            uint64_t k0, uint64_t k1) {
    const uint64_t M0 = 0xD2E7470EE14C6C93ULL, M1 = 0xCA5A826395121157ULL;
    const uint64_t W0 = 0x9E3779B97F4A7C15ULL, W1 = 0xBB67AE8584CAA73BULL;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t hi0 = __umul64hi(M0, c0), lo0 = M0 * c0;
        const uint64_t hi1 = __umul64hi(M1, c2), lo1 = M1 * c2;
        const uint64_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
        k0 += W0; k1 += W1;
    }
    U4 o; o.x[0] = c0; o.x[1] = c1; o.x[2] = c2; o.x[3] = c3;
    return o;
}

// Word q (0..3) of a block, chosen by selects: indexing r.x with a lane-varying
// q would put the block in a per-thread array, which the compiler moves to LDS
// and addresses through the dispatch packet, one host-memory read per wave at
// start-up (about 14 us of serialized reads for a 1000-wave launch).
__device__ __forceinline__ uint64_t philox_word(const U4& r, int q) {
    return q == 0 ? r.x[0] : q == 1 ? r.x[1] : q == 2 ? r.x[2] : r.x[3];
}

constexpr uint64_t MC_STREAM = 2;

// Uniform from one 64-bit word: top 53 bits / 2^53 (double), top 24 / 2^24 (float).
__device__ __forceinline__ double unif(uint64_t r, double) { return (double)(r >> 11) * 0x1.0p-53; }
__device__ __forceinline__ float unif(uint64_t r, float) { return (float)(uint32_t)(r >> 40) * 0x1.0p-24f; }

}  // namespace reach
