// common.h -- device helpers shared by the EBBkC HIP kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define EBB_WAVE 64

#define HIP_TRY(expr)                                  \
    do {                                               \
        hipError_t e_ = (expr);                        \
        if (e_ != hipSuccess) return EBBKC_E_HIP;      \
    } while (0)

namespace ebb {

__device__ __forceinline__ int lane_id() { return __lane_id(); }

__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }

// lanes strictly below this one
__device__ __forceinline__ uint64_t lanemask_lt() {
    return (lane_id() == 0) ? 0ull : (~0ull >> (64 - lane_id()));
}

__device__ __forceinline__ int popc64(uint64_t x) { return __popcll(x); }

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

template <typename T>
__device__ __forceinline__ T wave_min(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        T w = __shfl_xor(v, o, 64);
        v = w < v ? w : v;
    }
    return v;
}

template <typename T>
__device__ __forceinline__ T wave_max(T v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        T w = __shfl_xor(v, o, 64);
        v = w > v ? w : v;
    }
    return v;
}

// inclusive prefix sum across the wave
template <typename T>
__device__ __forceinline__ T wave_incl_scan(T v) {
    int l = lane_id();
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        T w = __shfl_up(v, o, 64);
        if (l >= o) v += w;
    }
    return v;
}

// Sum over the workgroup added to *out by one thread: a counter takes about
// 140 M atomics a second whatever their number of waves, so sums over many
// waves are folded per workgroup and their grids kept to a few hundred.  Every
// thread of the workgroup calls it; smem holds one value per wave.
template <typename T>
__device__ __forceinline__ void block_add(T v, T* smem, unsigned long long* out) {
    v = wave_sum(v);
    __syncthreads();
    if (lane_id() == 0) smem[threadIdx.x / EBB_WAVE] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (unsigned i = 1; i < blockDim.x / EBB_WAVE; ++i) v += smem[i];
        if (v) atomicAdd(out, (unsigned long long)v);
    }
}
constexpr unsigned SUM_GRID = 512;  // workgroups of a pass that ends in block_add

__device__ __forceinline__ int uniform_i32(int v) { return __builtin_amdgcn_readfirstlane(v); }

// of two indices from 0 on (their sum may pass 2^31)
__device__ __forceinline__ int midpoint(int lo, int hi) { return (int)(((unsigned)lo + (unsigned)hi) >> 1); }

// first index in sorted a[lo,hi) with a[i] >= key
__device__ __forceinline__ int lower_bound_i32(const int32_t* __restrict__ a, int lo, int hi, int32_t key) {
    while (lo < hi) {
        const int mid = midpoint(lo, hi);
        if (a[mid] < key) lo = mid + 1; else hi = mid;
    }
    return lo;
}

}  // namespace ebb
