// Coalesced transfers between global memory and the lane-owned registers of a
// window of 64 E cells: through LDS rows padded by 16 bytes, so that every
// global access is a 16-byte vector access although each lane owns E
// consecutive cells.  The rows belong to one wave; no other wave's data is
// read, so only the order of the wave's own LDS accesses has to hold.
#pragma once
#include "dev.hpp"

namespace reach {

// Order of one wave's LDS accesses for the compiler (the hardware keeps them in
// order): the waves of a block do not wait for each other.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 16 bytes of T: `type` 16-byte aligned (LDS rows), `any` aligned like T (global
// arrays: a workspace half or a caller's slice may start at any element; the
// hardware takes 16-byte accesses at any element address).
template <class T> struct Vec16;
template <> struct Vec16<double> {
    typedef double type __attribute__((ext_vector_type(2)));
    typedef double any __attribute__((ext_vector_type(2), aligned(8)));
};
template <> struct Vec16<float> {
    typedef float type __attribute__((ext_vector_type(4)));
    typedef float any __attribute__((ext_vector_type(4), aligned(4)));
};

template <class T, int E> struct TileIO {
    static constexpr int VEC = 16 / (int)sizeof(T);
    static constexpr bool STAGED = (E % VEC) == 0;
    static constexpr int ROW = E + VEC;
    static constexpr int LDS_ELEMS = STAGED ? WAVE * ROW : 1;
    using V = typename Vec16<T>::type;
    using G = typename Vec16<T>::any;

    template <bool NT>
    static __device__ __forceinline__ V ld(const T* p) {
        const G* q = reinterpret_cast<const G*>(p);
        if constexpr (NT) return __builtin_nontemporal_load(q);
        else return *q;
    }
    template <bool NT>
    static __device__ __forceinline__ void st(T* p, V v) {
        G* q = reinterpret_cast<G*>(p);
        if constexpr (NT) __builtin_nontemporal_store(v, q);
        else *q = v;
    }
    // the window's global reads into LDS rows (NT: non-temporal)
    template <bool NT>
    static __device__ __forceinline__ void gather(const T* __restrict__ src, int64_t ts, T* lds) {
        const int lane = threadIdx.x & (WAVE - 1);
#pragma unroll
        for (int j = 0; j < E / VEC; ++j) {
            const int el = (j * WAVE + lane) * VEC;
            const V v = ld<NT>(src + ts + el);
            *reinterpret_cast<V*>(lds + (el / E) * ROW + (el % E)) = v;
        }
    }
    // LDS rows to the window's global cells [olo, ohi) (NT: non-temporal)
    template <bool NT>
    static __device__ __forceinline__ void scatter(T* __restrict__ dst, int64_t ts, int olo, int ohi,
                                                   const T* lds) {
        const int lane = threadIdx.x & (WAVE - 1);
#pragma unroll
        for (int j = 0; j < E / VEC; ++j) {
            const int el = (j * WAVE + lane) * VEC;
            const V x = *reinterpret_cast<const V*>(lds + (el / E) * ROW + (el % E));
            if (el >= olo && el + VEC <= ohi) {
                st<NT>(dst + ts + el, x);
            } else {
#pragma unroll
                for (int q = 0; q < VEC; ++q)
                    if (el + q >= olo && el + q < ohi) dst[ts + el + q] = x[q];
            }
        }
    }

    // Cells [ts, ts + 64E) of src into lane registers; cells >= n get `ghost`.
    // `fast`: the window lies inside the chain; `nt`: its global accesses are
    // non-temporal.
    static __device__ __forceinline__ void load(T (&dst)[E], const T* __restrict__ src, int64_t ts,
                                                int64_t n, T ghost, bool fast, bool nt, T* lds) {
        const int lane = threadIdx.x & (WAVE - 1);
        if constexpr (STAGED) {
            if (fast) {
                constexpr int CPL = E / VEC;
                if (nt) gather<true>(src, ts, lds);
                else gather<false>(src, ts, lds);
                wave_sync();
#pragma unroll
                for (int j = 0; j < CPL; ++j) {
                    const V v = *reinterpret_cast<const V*>(lds + lane * ROW + j * VEC);
#pragma unroll
                    for (int q = 0; q < VEC; ++q) dst[j * VEC + q] = v[q];
                }
                wave_sync();
                return;
            }
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int64_t g = ts + (int64_t)lane * E + e;
            dst[e] = (g < n) ? src[g] : ghost;
        }
    }

    // Window cells [olo, ohi) of the lane registers to dst[ts + ...].
    static __device__ __forceinline__ void store(const T (&v)[E], T* __restrict__ dst, int64_t ts,
                                                 int olo, int ohi, bool fast, bool nt, T* lds) {
        const int lane = threadIdx.x & (WAVE - 1);
        if constexpr (STAGED) {
            if (fast) {
                constexpr int CPL = E / VEC;
#pragma unroll
                for (int j = 0; j < CPL; ++j) {
                    V x;
#pragma unroll
                    for (int q = 0; q < VEC; ++q) x[q] = v[j * VEC + q];
                    *reinterpret_cast<V*>(lds + lane * ROW + j * VEC) = x;
                }
                wave_sync();
                if (nt) scatter<true>(dst, ts, olo, ohi, lds);
                else scatter<false>(dst, ts, olo, ohi, lds);
                wave_sync();
                return;
            }
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int el = lane * E + e;
            if (el >= olo && el < ohi) dst[ts + el] = v[e];
        }
    }
};

template <class T> __device__ __forceinline__ SysPrm<T> make_prm(const double (&p)[5]) {
    SysPrm<T> P;
    P.a0 = (T)p[0]; P.a1 = (T)p[1]; P.a2 = (T)p[2]; P.a3 = (T)p[3]; P.a4 = (T)p[4];
    return P;
}

}  // namespace reach
