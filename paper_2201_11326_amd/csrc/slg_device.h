// Device helpers shared by the gfx950 kernels of more than one source file.
#pragma once

#include "slg_internal.h"
#include "slg_position.h"

namespace slg {
namespace {

// ---------------------------------------------------------------------------
// wavefront / workgroup primitives
// ---------------------------------------------------------------------------
__device__ __forceinline__ int lane_id() { return __lane_id(); }

// Pointers that reach a kernel through LDS or a struct in memory lose their
// address space; naming it keeps their accesses global_* (flat accesses also
// count against the LDS wait counter, so every LDS wait would wait for them).
template <typename T>
__device__ __forceinline__ __attribute__((address_space(1))) T *as_global(T *p) {
    return (__attribute__((address_space(1))) T *)p;
}

// Wavefront-uniform values moved to scalar registers.
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ long long uniform(long long x) {
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(x & 0xFFFFFFFFll));
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)((unsigned long long)x >> 32));
    return (long long)(((unsigned long long)hi << 32) | lo);
}
template <typename T>
__device__ __forceinline__ T *uniform(T *p) {
    return reinterpret_cast<T *>(uniform((long long)reinterpret_cast<uintptr_t>(p)));
}

__device__ __forceinline__ int bits_below(unsigned long long mask) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}

// LDS writes of this wavefront become visible to its other lanes.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename T>
__device__ __forceinline__ T wave_sum(T x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

__device__ __forceinline__ int wave_max(int x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x = max(x, __shfl_xor(x, o));
    return x;
}

template <typename T>
__device__ __forceinline__ T wave_incl_scan(T x) {
    const int lane = lane_id();
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        T y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    return x;
}

// Exclusive scan over a workgroup of NT threads; `wsum` holds NT/64 entries.
template <int NT, typename T>
__device__ __forceinline__ T block_excl_scan(T x, T *wsum, T &total) {
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    T incl = wave_incl_scan(x);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    T pre = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
        T t = wsum[w];
        pre += (w < wave) ? t : T(0);
        tot += t;
    }
    total = tot;
    __syncthreads();
    return pre + incl - x;
}

// As block_excl_scan, without the trailing barrier: the caller guarantees
// a workgroup barrier before `wsum` is written again.
template <int NT, typename T>
__device__ __forceinline__ T block_excl_scan_open(T x, T *wsum, T &total) {
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    T incl = wave_incl_scan(x);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    T pre = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
        T t = wsum[w];
        pre += (w < wave) ? t : T(0);
        tot += t;
    }
    total = tot;
    return pre + incl - x;
}

// Copy the by-value parameter block into LDS, one dword per thread (the
// caller follows with a workgroup barrier).
__device__ __forceinline__ void stage_params(EmitParams *dst, const EmitParams &src) {
    constexpr int kWords = (int)(sizeof(EmitParams) / 4);
    static_assert(sizeof(EmitParams) % 4 == 0, "EmitParams is dword-sized");
    const int32_t *from = reinterpret_cast<const int32_t *>(&src);
    int32_t *to = reinterpret_cast<int32_t *>(dst);
    for (int x = threadIdx.x; x < kWords; x += blockDim.x) to[x] = from[x];
}

// First position in a[lo, hi) holding a value >= key (a sorted ascending).
__device__ __forceinline__ int lower_bound_i32(const int32_t *__restrict__ a, int lo, int hi,
                                               int key) {
    while (lo < hi) {
        const int mid = middle(lo, hi);
        if (a[mid] < key)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

}  // namespace
}  // namespace slg
