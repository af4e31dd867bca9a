// Many small embedding queries on gfx950: offline batches and online serving.
//
// Every query (FP64, n <= 512 cells, scalar input) is run by one wavefront
// with its whole lower/upper state in registers (E = ceil(n / 64) cells per
// lane, 1..8, spread so that every lane is busy), all N RK4 steps in one go:
// no halo, no HBM traffic inside the step loop.  Long cooperative queries, and
// served ones, take a wavefront per side; the queries of a large batch share
// wavefronts at 2 to 16 cells per lane.  The arithmetic per cell is the
// large-n embedding kernel's, so a query gives the same box alone, in a batch,
// or served.
//
//   batch_kernel   persistent grid; each wave pops the next work item (a query, or
//                  one side of the longest cooperative ones) from a device
//                  counter until the batch is exhausted.
//   pack_kernel    the same for a packed batch, whose items are segment packs:
//                  queries sharing a wave at E cells per lane
//                  (pack_sides_kernel: the longest of them one side per wave).
//   single_kernel  one query per launch (the baseline the batch is compared with).
//   serve_kernel   persistent grid fed through a ring of descriptors in pinned
//                  host memory; each wave claims the next work item (sequence
//                  number and side), waits (bounded) until the host publishes
//                  it, runs it and publishes that side's completion.  The grid
//                  leaves as a whole when the host sets the stop flag or when
//                  any wave reaches the idle limit, so it always drains.  A
//                  served query reads its host-written cancel word every
//                  kCancelEvery steps and stops early when it is set.
#include "batch_pack.hpp"

namespace reach {

// Cancel word of the queries that have none (batches, single launches).
__device__ unsigned int g_never_cancelled = 0u;

// One query, or one side of it: S = 2 runs both sides in this wave, S = 1
// only side `side` (cooperative systems, whose sides do not interact).
template <int KIND, int E, int S>
__device__ __noinline__ unsigned run_query_E(const QDesc& d, int side) {
    using T = double;
    const int64_t n = d.n;
    const Lanes L = lanes_of<E>(n);
    const double* src[2] = {d.x_lo, d.x_hi};
    double* dst[2] = {d.r_lo, d.r_hi};
    const double* pin[2] = {d.p_lo, d.p_hi};
    T y[S][E];
    Inputs<T, E, S, IN_SCALAR> U;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const int sd = S == 1 ? side : s;
#pragma unroll
        for (int e = 0; e < E; ++e)
            y[s][e] = (e < L.cnt) ? src[sd][L.first + e] : ghost<KIND, T>();
        U.u[s] = pin[sd] ? *pin[sd] : T(0);
    }
    SysPrm<T> P;
    P.a0 = d.prm[0]; P.a1 = d.prm[1]; P.a2 = d.prm[2]; P.a3 = d.prm[3]; P.a4 = d.prm[4];
    const Steps<T> st = {d.h2, d.dt, d.dt6};
    T acc[S][E], t[S][E];
    // Steps in blocks of kCancelEvery.  A served query reads its cancel word
    // at the start of a block and looks at the value only after the block's
    // steps, so the host-memory read never stalls the arithmetic.  Queries
    // without one read a device word that is always 0 (no branch around the
    // load, so nothing has to wait for it before the steps).
    const unsigned int* cw = d.cancel ? d.cancel : &g_never_cancelled;
    bool cancelled = false;
    for (int64_t k0 = 0; k0 < d.nsteps; k0 += kCancelEvery) {
        const unsigned stop = __hip_atomic_load(cw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        const int64_t k1 = k0 + kCancelEvery < d.nsteps ? k0 + kCancelEvery : d.nsteps;
        for (int64_t k = k0; k < k1; ++k) {
            bal_stage<KIND, 1, E, S>(y, acc, t, P, U, st, L);
            bal_stage<KIND, 2, E, S>(y, acc, t, P, U, st, L);
            bal_stage<KIND, 3, E, S>(y, acc, t, P, U, st, L);
            bal_stage<KIND, 4, E, S>(y, acc, t, P, U, st, L);
        }
        if (wave_bcast(stop)) {
            cancelled = true;
            break;
        }
    }
    if (cancelled) return ST_CANCELLED;
    unsigned bits = 0;
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
    const unsigned long long nf = __ballot(bits & ST_NONFINITE);
    const unsigned long long od = __ballot(bits & ST_ORDER);
    return (nf ? (unsigned)ST_NONFINITE : 0u) | (od ? (unsigned)ST_ORDER : 0u);
}

template <int KIND, int S>
__device__ __forceinline__ unsigned run_query_kind(const QDesc& d, int side) {
    switch (d.E) {
        case 1: return run_query_E<KIND, 1, S>(d, side);
        case 2: return run_query_E<KIND, 2, S>(d, side);
        case 3: return run_query_E<KIND, 3, S>(d, side);
        case 4: return run_query_E<KIND, 4, S>(d, side);
        case 5: return run_query_E<KIND, 5, S>(d, side);
        case 6: return run_query_E<KIND, 6, S>(d, side);
        case 7: return run_query_E<KIND, 7, S>(d, side);
        default: return run_query_E<KIND, 8, S>(d, side);
    }
}

// Whole query in one wave (descriptor fields are wave-uniform; the host
// validated kind and E).
__device__ __forceinline__ unsigned run_query(const QDesc& d) {
    if (d.kind == K_CTM) return run_query_kind<K_CTM, 2>(d, 0);
    if (d.kind == K_RD) return run_query_kind<K_RD, 2>(d, 0);
    return run_query_kind<K_LIN3, 2>(d, 0);
}

// Work item (query, side).  Cooperative queries split into two waves, one per
// side, which halves the dependent chain of a query; the coupled LIN3 query
// runs whole in its side-0 item and its side-1 item is empty.
__device__ __forceinline__ bool item_is_empty(const QDesc& d, int side) {
    return d.kind == K_LIN3 && side == 1;
}
__device__ __forceinline__ bool item_is_whole(const QDesc& d) { return d.kind == K_LIN3; }
__device__ __forceinline__ unsigned run_item(const QDesc& d, int side) {
    if (d.kind == K_CTM) return run_query_kind<K_CTM, 1>(d, side);
    if (d.kind == K_RD) return run_query_kind<K_RD, 1>(d, side);
    return run_query_kind<K_LIN3, 2>(d, 0);
}

// lower > upper check of a finished query, by the wave that finished last
__device__ __forceinline__ unsigned order_bits(const QDesc& d) {
    unsigned bits = 0;
    for (int64_t j = threadIdx.x; j < d.n; j += WAVE)
        if (d.r_lo[j] > d.r_hi[j]) bits = ST_ORDER;
    return __ballot(bits) ? (unsigned)ST_ORDER : 0u;
}

__global__ __launch_bounds__(64) void batch_kernel(const QDesc* __restrict__ desc,
                                                   const BatchItem* __restrict__ items,
                                                   const uint32_t* __restrict__ members,
                                                   const uint64_t* n_items,
                                                   unsigned long long* counter,
                                                   unsigned int* qflags, unsigned int* pair,
                                                   unsigned int* status) {
    const int lane = threadIdx.x;
    const uint64_t nw = wave_bcast(*n_items);
    const uint64_t ni = nw & 0xFFFFFFFFu, ns = nw >> 32;
    for (;;) {
        uint64_t u = 0;
        if (lane == 0) u = atomicAdd(counter, 1ULL);
        u = wave_bcast(u);
        if (u >= ni + ns) break;
        // one side of item u / 2, or the whole of a shorter query (4000 CTM and RD queries of
        // 100 steps: 200 us whole, 490 by sides, which wait for each other's results
        // through memory; 2000 of 10 to 1000 steps, the longest by sides: 470 for 950)
        const bool one = u < 2 * ns;
        const uint64_t i = one ? u >> 1 : u - ns;
        const int side = one ? (int)(u & 1) : 0;
        const QDesc d = desc[members[items[i].start]];
        if (item_is_empty(d, side)) continue;
        unsigned bits = one ? run_item(d, side) : run_query(d);
        if (one && !item_is_whole(d)) {
            // publish this side, then the second side to finish checks the order
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            uint64_t old = 0;
            if (lane == 0)
                old = __hip_atomic_fetch_add(&pair[i], 1u, __ATOMIC_ACQ_REL,
                                             __HIP_MEMORY_SCOPE_AGENT);
            old = wave_bcast(old);
            if (old == 1) {
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                bits |= order_bits(d);
            }
        }
        if (lane == 0 && bits) {
            atomicOr(&qflags[d.tag], bits);
            atomicOr(status, bits);
        }
    }
}

__global__ __launch_bounds__(64) void single_kernel(QDesc d, unsigned int* status,
                                                    unsigned int* flags) {
    const unsigned bits = run_query(d);
    if (threadIdx.x == 0) {
        if (flags) *flags = bits;
        else if (bits) atomicOr(status, bits);
    }
}

__global__ __launch_bounds__(256) void zero_kernel(unsigned int* p, int64_t count) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0u;
}

// A served item's box arrives in pinned host staging; the wave that runs it
// copies what it reads (its side, or both sides of a coupled LIN3 query) into
// the query's device pool block, points its copy of the descriptor there, and
// runs from it.  The fences make the lanes' stores visible to the wave's own
// loads of other lanes' cells (agent-scope release, then acquire: the vector
// L1 may hold the block from an earlier query).
__device__ __forceinline__ void park_box(QDesc& d, int side) {
    const int lane = threadIdx.x;
    const int64_t n = d.n;
    double* blk = d.park;
    const bool both = item_is_whole(d);
    for (int s = 0; s < 2; ++s) {
        if (!both && s != side) continue;
        const double* src = s ? d.x_hi : d.x_lo;
        double* dst = blk + (int64_t)s * n;
        for (int64_t j = lane; j < n; j += WAVE) dst[j] = src[j];
        if (d.p_lo && lane == 0) blk[2 * n + s] = s ? *d.p_hi : *d.p_lo;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    d.x_lo = blk;
    d.x_hi = blk + n;
    if (d.p_lo) {
        d.p_lo = blk + 2 * n;
        d.p_hi = blk + 2 * n + 1;
    }
}

// ctl[0]: claim counter (work items: two per sequence number, one per side),
// ctl[1]: status bits, ctl[2]: watermark (every sequence below it has been
// seen published), ctl[3]: grid quit word.  Only the waves holding the
// sequence at the watermark read the host ring; the others wait on device
// memory, so idle waves do not flood the host link with polls.  The first wave
// to reach the idle limit sets the quit word, and every other wave leaves at
// its next wait iteration or claim: the grid exits as a whole, and the host
// moves any query published to a sequence no wave will run to a new grid.
__global__ __launch_bounds__(64) void serve_kernel(ServeSlot* ring, int32_t slots,
                                                   unsigned long long* ctl,
                                                   volatile unsigned int* stop,
                                                   unsigned int* status, int64_t idle_cycles) {
    const int lane = threadIdx.x;
    unsigned long long* claim = ctl;
    unsigned long long* seen = ctl + 2;
    unsigned long long* quitw = ctl + 3;
    for (;;) {
        uint64_t u = 0, gq = 0;
        if (lane == 0) {
            gq = __hip_atomic_load(quitw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (!gq) u = atomicAdd(claim, 1ULL);
        }
        if (wave_bcast(gq)) return;
        u = wave_bcast(u);
        const uint64_t t = u >> 1;
        const int side = (int)(u & 1);
        ServeSlot* sl = &ring[t % (uint64_t)slots];
        // Wait until the host publishes sequence t in this slot, the host asks
        // to stop, another wave ends the grid, or the idle limit passes.
        // Every branch ends the wait.
        const uint64_t t_start = wall_clock64();
        int quit = 0;
        for (uint32_t it = 0;; ++it) {
            uint64_t seq = 0, w = 0, q = 0;
            unsigned st = 0;
            if (lane == 0) {
                w = __hip_atomic_load(seen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                q = __hip_atomic_load(quitw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (w >= t)
                    seq = __hip_atomic_load(&sl->seq, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_SYSTEM);
                if ((it & 63u) == 0u)
                    st = __hip_atomic_load((unsigned int*)stop, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_SYSTEM);
            }
            seq = wave_bcast(seq);
            w = wave_bcast(w);
            q = wave_bcast(q);
            st = (unsigned)wave_bcast(st);
            if (seq == t + 1) break;
            if (st || q) { quit = 1; break; }
            if ((int64_t)(wall_clock64() - t_start) > idle_cycles) {
                if (lane == 0)
                    __hip_atomic_store(quitw, 1ULL, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                quit = 1;
                break;
            }
            if (w >= t) __builtin_amdgcn_s_sleep(2);
            else __builtin_amdgcn_s_sleep(32);
        }
        if (quit) return;
        if (lane == 0) atomicMax(seen, (unsigned long long)(t + 1));
        __atomic_thread_fence(__ATOMIC_ACQUIRE);
        QDesc d = sl->d;
        const bool empty = item_is_empty(d, side);
        if (d.park && !empty) park_box(d, side);
        const unsigned bits = empty ? 0u : run_item(d, side);
        if (lane == 0) {
            sl->flags[side] = bits;
            if (bits & (ST_NONFINITE | ST_ORDER)) atomicOr(status, bits & (ST_NONFINITE | ST_ORDER));
            __hip_atomic_store(&sl->done[side], t + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

// The packed batch whose longest items run one side per wave (batch_sides.hip).
// pack_kernel keeps its own signature: with one more argument the compiler
// allocates the same instructions' registers differently, and 10^5 queries take
// 2.5% longer.
hipError_t launch_pack_sides(const QDesc* d, const BatchItem* items, const uint32_t* members,
                             const uint64_t* n_items, unsigned long long* counter,
                             unsigned int* qflags, unsigned int* pair, unsigned int* status,
                             bool wide, int64_t grid, hipStream_t s);

hipError_t launch_batch(const QDesc* d, const BatchItem* items, const uint32_t* members,
                        const uint64_t* n_items, unsigned long long* counter,
                        unsigned int* qflags, unsigned int* pair, unsigned int* status,
                        bool sides, int packed, int64_t grid, hipStream_t s) {
    if (packed && sides)
        return launch_pack_sides(d, items, members, n_items, counter, qflags, pair, status,
                                 packed == 2, grid, s);
    if (packed == 2)
        hipLaunchKernelGGL(pack_kernel<16>, dim3((unsigned)grid), dim3(WAVE), 0, s, d, items,
                           members, n_items, counter, qflags, status);
    else if (packed)
        hipLaunchKernelGGL(pack_kernel<8>, dim3((unsigned)grid), dim3(WAVE), 0, s, d, items,
                           members, n_items, counter, qflags, status);
    else
        hipLaunchKernelGGL(batch_kernel, dim3((unsigned)grid), dim3(WAVE), 0, s, d, items,
                           members, n_items, counter, qflags, pair, status);
    return hipGetLastError();
}

hipError_t launch_single(const QDesc& d, unsigned int* status, unsigned int* flags,
                         hipStream_t s) {
    hipLaunchKernelGGL(single_kernel, dim3(1), dim3(WAVE), 0, s, d, status, flags);
    return hipGetLastError();
}

hipError_t launch_zero(void* p, int64_t count, hipStream_t s) {
    const unsigned grid = (unsigned)((count + 255) / 256);
    hipLaunchKernelGGL(zero_kernel, dim3(grid > 0 ? grid : 1), dim3(256), 0, s,
                       (unsigned int*)p, count);
    return hipGetLastError();
}

hipError_t launch_server(ServeSlot* ring, int32_t slots, unsigned long long* ctl,
                         volatile unsigned int* stop, unsigned int* status, int64_t idle_cycles,
                         int64_t grid, hipStream_t s) {
    hipLaunchKernelGGL(serve_kernel, dim3((unsigned)grid), dim3(WAVE), 0, s, ring, slots, ctl,
                       stop, status, idle_cycles);
    return hipGetLastError();
}

}  // namespace reach
