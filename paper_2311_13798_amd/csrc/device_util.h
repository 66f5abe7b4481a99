// device_util.h -- wave-level helpers for the bitmap kernels (wave64).
#pragma once
#include "arena.h"
#include "common.h"

namespace ebb {

// Order this wave's LDS accesses: everything before is visible to every lane after.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Words that several workgroups exchange while a kernel runs: relaxed
// device-scope accesses, which go past the compute units' vector caches and the
// L2s of the eight dies.  Order between them comes from waiting for one before
// the next is issued (wait_memory, or the use of a returned value); release and
// acquire would write back and drop whole caches instead.
template <typename T>
__device__ __forceinline__ T dev_load(const T* p) {
    return __hip_atomic_load(const_cast<T*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void dev_store(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T dev_add(T* p, T v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// the wave's loads have returned and its stores and atomics are done
__device__ __forceinline__ void wait_memory() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory"); }

// a wave-uniform 64-bit value in scalar registers
__device__ __forceinline__ uint64_t uni64(uint64_t x) {
    uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
    uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// Wave64 reductions of 32-bit values: DPP moves within each row of 16 lanes
// (swap neighbours, swap pairs, mirror within 8, mirror within 16), then the
// four row results read into scalars.  Every lane of the wave must be active.
template <int CTRL>
__device__ __forceinline__ int dpp_mov(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
enum : int { DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_MIRROR = 0x140 };

__device__ __forceinline__ uint32_t wsum_u32(uint32_t v) {
    int x = (int)v;
    x += dpp_mov<DPP_XOR1>(x);
    x += dpp_mov<DPP_XOR2>(x);
    x += dpp_mov<DPP_HALF_MIRROR>(x);
    x += dpp_mov<DPP_MIRROR>(x);
    return (uint32_t)__builtin_amdgcn_readlane(x, 0) + (uint32_t)__builtin_amdgcn_readlane(x, 16) +
           (uint32_t)__builtin_amdgcn_readlane(x, 32) + (uint32_t)__builtin_amdgcn_readlane(x, 48);
}

__device__ __forceinline__ int wmax_i32(int x) {
    x = max(x, dpp_mov<DPP_XOR1>(x));
    x = max(x, dpp_mov<DPP_XOR2>(x));
    x = max(x, dpp_mov<DPP_HALF_MIRROR>(x));
    x = max(x, dpp_mov<DPP_MIRROR>(x));
    return max(max(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
               max(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}

__device__ __forceinline__ int wmin_i32(int x) {
    x = min(x, dpp_mov<DPP_XOR1>(x));
    x = min(x, dpp_mov<DPP_XOR2>(x));
    x = min(x, dpp_mov<DPP_HALF_MIRROR>(x));
    x = min(x, dpp_mov<DPP_MIRROR>(x));
    return min(min(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
               min(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}

// Transpose of a 64 x 64 bit matrix held one row per lane: lane i gets the
// bits i of all lanes, lane j's at position j (blocks swapped across lanes
// lane ^ 32, ^ 16, .. ^ 1).  Every lane must be active.
__device__ __forceinline__ uint64_t transpose64(uint64_t x) {
    const int lane = lane_id();
    constexpr uint64_t M[6] = {0x00000000FFFFFFFFull, 0x0000FFFF0000FFFFull, 0x00FF00FF00FF00FFull,
                               0x0F0F0F0F0F0F0F0Full, 0x3333333333333333ull, 0x5555555555555555ull};
#pragma unroll
    for (int b = 0; b < 6; ++b) {
        const int s = 32 >> b;
        const uint64_t y = __shfl_xor(x, s, 64);
        x = (lane & s) ? (x & ~M[b]) | ((y >> s) & M[b]) : (x & M[b]) | ((y << s) & ~M[b]);
    }
    return x;
}

// bits strictly above x within word w of a multi-word row
__device__ __forceinline__ uint64_t upper_mask(int x, int w) {
    int xw = x >> 6, xb = x & 63;
    if (w < xw) return 0;
    if (w > xw) return ~0ull;
    return xb == 63 ? 0ull : (~0ull << (xb + 1));
}

template <int W>
__device__ __forceinline__ int popcW(const uint64_t (&p)[W]) {
    int c = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) c += popc64(p[w]);
    return c;
}

// rows [0, c) as a W-word mask
template <int W>
__device__ __forceinline__ void prefix_mask(int c, uint64_t (&p)[W]) {
#pragma unroll
    for (int w = 0; w < W; ++w) {
        int lo = 64 * w;
        p[w] = c >= lo + 64 ? ~0ull : (c > lo ? ((1ull << (c - lo)) - 1) : 0ull);
    }
}

// The items a wave draws from a launch's Tickets (arena.h); every value is
// wave-uniform.
struct Drawn {
    int64_t cur = 0, left = 0, step = 0;
    bool started = false;
    // the next item, or -1 when none is left
    __device__ __forceinline__ int64_t next(const Tickets& T) {
        if (left == 0) {
            const int64_t waves = T.dealt ? (int64_t)gridDim.x * (blockDim.x / EBB_WAVE) : 0;
            const int64_t total = T.heavy + T.nchunks;
            uint64_t t;
            if (!started && T.dealt) {
                const uint64_t wave = threadIdx.x / EBB_WAVE, per = blockDim.x / EBB_WAVE;
                t = T.dealt == 2 ? blockIdx.x * per + wave : wave * gridDim.x + blockIdx.x;
                started = true;
            } else {
                if (total <= waves) return -1;
                t = 0;
                if (lane_id() == 0) t = waves + atomicAdd(T.next, 1ull);
            }
            t = uni64(t);
            if ((int64_t)t >= total) return -1;
            if ((int64_t)t < T.heavy) {
                cur = t;
                left = 1;
                step = 0;
            } else if (T.chunk_len > 0) {
                cur = T.heavy + ((int64_t)t - T.heavy) * T.chunk_len;
                left = T.n - cur < T.chunk_len ? T.n - cur : T.chunk_len;
                step = 1;
            } else {
                const int64_t j = (int64_t)t - T.heavy;
                cur = T.heavy + j;
                left = (T.n - T.heavy - j + T.nchunks - 1) / T.nchunks;
                step = T.nchunks;
            }
        }
        const int64_t it = cur;
        cur += step;
        --left;
        return it;
    }
};

// Tickets of n items for a launch of `waves` waves: every light item dealt to
// one chunk per wave when nothing heavy comes first (then no wave touches the
// counter), else two per wave, since the waves come to them at different times.
// consecutive > 0: chunks of up to that many neighbours, sixteen or more per wave.
// once: a launch that is not persistent, each wave drawing once; a workgroup
// leaves with its slowest wave, so its waves take neighbours, which weigh alike
// (Chung-Lu 3e5 at k = 10 135 ms, against 249 with one task of each quarter of
// the list; a persistent launch puts neighbours, heavy ones first, on different
// compute units).
inline Tickets make_tickets(unsigned long long* next, int64_t n, int64_t heavy, int64_t waves, int consecutive,
                            bool shared, bool once = false) {
    Tickets T{next, n, heavy < n ? heavy : n, 0, 0, shared ? 0 : (once ? 2 : 1)};
    const int64_t light = T.n - T.heavy;
    if (consecutive > 0) {
        int64_t len = light / (16 * waves);
        len = len < 1 ? 1 : (len > consecutive ? consecutive : len);
        T.chunk_len = (int32_t)len;
        T.nchunks = (light + len - 1) / len;
    } else {
        const int64_t most = T.heavy ? 2 * waves : waves;
        T.nchunks = light < most ? light : most;
    }
    return T;
}

}  // namespace ebb
