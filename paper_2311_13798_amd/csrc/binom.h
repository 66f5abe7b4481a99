// binom.h -- binomial tables and exact 128-bit arithmetic for the closed forms.
// Every source that includes this has tables of its own, filled by
// launch_tables there.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ebb {
namespace {

typedef unsigned __int128 u128;

// C(n, r) for n < BIN_N, r < BIN_R, saturated to UINT64_MAX when it does not fit
constexpr int BIN_N = 258, BIN_R = 65;
__device__ uint64_t g_binom[BIN_N * BIN_R];

// C(n, r) or UINT64_MAX if it does not fit 64 bits
__device__ uint64_t binom(int n, int r) {
    if (r < 0 || r > n) return 0;
    if (r > n - r) r = n - r;
    if (n < BIN_N && r < BIN_R) return g_binom[n * BIN_R + r];
    unsigned __int128 c = 1;
    for (int j = 1; j <= r; ++j) {
        c = c * (unsigned __int128)(n - r + j) / (unsigned __int128)j;
        if (c > (unsigned __int128)UINT64_MAX) return UINT64_MAX;
    }
    return (uint64_t)c;
}

// C(n, r) for n <= 257, r <= 128 in 128 bits (Pascal's rule, built once per
// device); both words all ones when it does not fit
constexpr int B128_N = 258, B128_R = 129;
__device__ uint64_t g_binom128[B128_N * B128_R * 2];

// Pascal's rule row by row in one workgroup: thread r owns column r and reads
// its left neighbour's value of the row before from LDS.  (One thread for the
// whole 128-bit table took 8.3 ms of every process's first count.)
__global__ void k_binom_init() {
    __shared__ u128 row[2][B128_R];
    __shared__ bool sat[2][B128_R];
    const int r = threadIdx.x;
    for (int n = 0; n < B128_N; ++n) {
        const int cur = n & 1, old = cur ^ 1;
        if (r < B128_R) {
            u128 v = r == 0 ? 1 : 0;
            bool s = false;
            if (r > 0 && r <= n) {
                const u128 x = row[old][r - 1];
                v = x + row[old][r];
                s = sat[old][r - 1] || sat[old][r] || v < x;
            }
            row[cur][r] = v;
            sat[cur][r] = s;
            uint64_t* o = &g_binom128[(n * B128_R + r) * 2];
            o[0] = s ? ~0ull : (uint64_t)v;
            o[1] = s ? ~0ull : (uint64_t)(v >> 64);
            if (r < BIN_R) g_binom[n * BIN_R + r] = s || (v >> 64) ? UINT64_MAX : (uint64_t)v;
        }
        __syncthreads();
    }
}
static_assert(BIN_N == B128_N && BIN_R <= B128_R, "one pass fills both tables");

// C(n, r) exactly in 128 bits; sets ovf when it does not fit
__device__ __forceinline__ u128 binom128(int n, int r, bool& ovf) {
    if (r < 0 || r > n) return 0;
    if (r > n - r) r = n - r;
    if (r == 0) return 1;
    if (n >= B128_N) { ovf = true; return 0; }
    const uint64_t* e = &g_binom128[(n * B128_R + r) * 2];
    const uint64_t lo = e[0], hi = e[1];
    if (lo == ~0ull && hi == ~0ull) { ovf = true; return 0; }
    return ((u128)hi << 64) | lo;
}

// a * b in 128 bits; sets ovf when it does not fit
__device__ __forceinline__ u128 mul128(u128 a, u128 b, bool& ovf) {
    const uint64_t ah = (uint64_t)(a >> 64), al = (uint64_t)a, bh = (uint64_t)(b >> 64), bl = (uint64_t)b;
    if (ah && bh) { ovf = true; return 0; }
    const u128 low = (u128)al * bl;
    const u128 mid = (u128)ah * bl + (u128)al * bh;  // one of the two terms is zero
    if (mid >> 64) { ovf = true; return 0; }
    const u128 r = low + (mid << 64);
    if (r < low) { ovf = true; return 0; }
    return r;
}

inline hipError_t launch_tables(hipStream_t s) {
    hipLaunchKernelGGL(k_binom_init, dim3(1), dim3(192), 0, s);
    return hipGetLastError();
}

}  // namespace
}  // namespace ebb
