// prims.hip -- exclusive scan and stable LSD radix sort (wave64, gfx950).
#include <algorithm>

#include "common.h"
#include "prims.h"

namespace ebb {

namespace {

constexpr int SCAN_BLOCK = 256;
constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_TILE = SCAN_BLOCK * SCAN_ITEMS;

__device__ __forceinline__ int64_t block_excl_scan(int64_t v, int64_t* total) {
    __shared__ int64_t wsum[SCAN_BLOCK / EBB_WAVE];
    int lane = lane_id(), w = threadIdx.x / EBB_WAVE;
    int64_t inc = wave_incl_scan(v);
    if (lane == EBB_WAVE - 1) wsum[w] = inc;
    __syncthreads();
    int64_t before = 0, all = 0;
#pragma unroll
    for (int i = 0; i < SCAN_BLOCK / EBB_WAVE; ++i) {
        if (i < w) before += wsum[i];
        all += wsum[i];
    }
    __syncthreads();
    *total = all;
    return before + inc - v;
}

template <typename T>
__global__ void k_tile_sums(const T* __restrict__ in, int64_t n, int64_t* __restrict__ part) {
    int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
    int64_t acc = 0;
#pragma unroll
    for (int j = 0; j < SCAN_ITEMS; ++j) {
        int64_t i = base + j * SCAN_BLOCK + threadIdx.x;
        if (i < n) acc += (int64_t)in[i];
    }
    acc = wave_sum(acc);
    __shared__ int64_t ws[SCAN_BLOCK / EBB_WAVE];
    if (lane_id() == 0) ws[threadIdx.x / EBB_WAVE] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t t = 0;
        for (int i = 0; i < SCAN_BLOCK / EBB_WAVE; ++i) t += ws[i];
        part[blockIdx.x] = t;
    }
}

// one block scans the tile sums in place (any count)
__global__ void k_scan_parts(int64_t* __restrict__ part, int64_t np, int64_t* __restrict__ d_total) {
    __shared__ int64_t carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int64_t base = 0; base < np; base += SCAN_BLOCK) {
        int64_t i = base + threadIdx.x;
        int64_t v = i < np ? part[i] : 0;
        int64_t tot;
        int64_t ex = block_excl_scan(v, &tot);
        if (i < np) part[i] = carry + ex;
        __syncthreads();
        if (threadIdx.x == 0) carry += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0 && d_total) *d_total = carry;
}

template <typename T>
__global__ void k_tile_scan(const T* __restrict__ in, int64_t* __restrict__ out, int64_t n,
                            const int64_t* __restrict__ part) {
    int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
    // each thread owns SCAN_ITEMS consecutive elements
    int64_t first = base + (int64_t)threadIdx.x * SCAN_ITEMS;
    int64_t v[SCAN_ITEMS];
    int64_t s = 0;
#pragma unroll
    for (int j = 0; j < SCAN_ITEMS; ++j) {
        int64_t i = first + j;
        v[j] = i < n ? (int64_t)in[i] : 0;
        s += v[j];
    }
    int64_t tot;
    int64_t ex = block_excl_scan(s, &tot) + part[blockIdx.x];
#pragma unroll
    for (int j = 0; j < SCAN_ITEMS; ++j) {
        int64_t i = first + j;
        if (i < n) out[i] = ex;
        ex += v[j];
    }
}

template <typename T>
hipError_t scan_impl(const T* in, int64_t* out, int64_t n, int64_t* d_total, int64_t* tmp, hipStream_t s) {
    if (n <= 0) {
        if (d_total) return hipMemsetAsync(d_total, 0, sizeof(int64_t), s);
        return hipSuccess;
    }
    int64_t nb = (n + SCAN_TILE - 1) / SCAN_TILE;
    hipLaunchKernelGGL(k_tile_sums<T>, dim3((unsigned)nb), dim3(SCAN_BLOCK), 0, s, in, n, tmp);
    hipLaunchKernelGGL(k_scan_parts, dim3(1), dim3(SCAN_BLOCK), 0, s, tmp, nb, d_total);
    hipLaunchKernelGGL(k_tile_scan<T>, dim3((unsigned)nb), dim3(SCAN_BLOCK), 0, s, in, out, n, tmp);
    return hipGetLastError();
}

// ---------------------------------------------------------------- radix sort
constexpr int RS_BLOCK = 256;
// Items a thread takes one after the other, each with four barriers: 16 keep
// the histograms small, 4 keep a short sort short (40,000 items: 20 us a
// scatter with 16, which is ten workgroups).
constexpr int RS_ITEMS = 16, RS_ITEMS_SHORT = 4;
constexpr int64_t RS_SHORT_N = 1 << 20;
inline bool rs_short(int64_t n, bool small_hist) { return n <= RS_SHORT_N && !small_hist; }
inline int64_t rs_blocks(int64_t n, bool small_hist = false) {
    const int64_t tile = RS_BLOCK * (rs_short(n, small_hist) ? RS_ITEMS_SHORT : RS_ITEMS);
    return (n + tile - 1) / tile;
}
constexpr int RS_WAVES = RS_BLOCK / EBB_WAVE;

template <typename K, int RS_ITEMS>
__global__ void k_rs_hist(const K* __restrict__ keys, int64_t n, int shift, int64_t nb,
                          int64_t* __restrict__ hist) {
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    int64_t base = (int64_t)blockIdx.x * (RS_BLOCK * RS_ITEMS);
    for (int j = 0; j < RS_ITEMS; ++j) {
        int64_t i = base + j * RS_BLOCK + threadIdx.x;
        if (i < n) atomicAdd(&h[(keys[i] >> shift) & 0xFF], 1u);
    }
    __syncthreads();
    hist[(int64_t)threadIdx.x * nb + blockIdx.x] = h[threadIdx.x];
}

// vin null: an item's value is its index; kout / vout null: not written
template <typename K, int RS_ITEMS>
__global__ void k_rs_scatter(const K* __restrict__ kin, const uint32_t* __restrict__ vin,
                             K* __restrict__ kout, uint32_t* __restrict__ vout, int64_t n, int shift,
                             int64_t nb, const int64_t* __restrict__ off) {
    __shared__ uint32_t run[256];
    __shared__ uint32_t wcnt[RS_WAVES][256];
    const int tid = threadIdx.x, lane = lane_id(), w = tid / EBB_WAVE;
    run[tid] = 0;
    int64_t base = (int64_t)blockIdx.x * (RS_BLOCK * RS_ITEMS);
    for (int j = 0; j < RS_ITEMS; ++j) {
        int64_t i = base + j * RS_BLOCK + tid;
        bool valid = i < n;
        K key = valid ? kin[i] : 0;
        uint32_t val = !valid ? 0 : (vin ? vin[i] : (uint32_t)i);
        int d = (int)((key >> shift) & 0xFF);
        uint64_t peers = ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            uint64_t bb = ballot(valid && ((d >> b) & 1));
            peers &= ((d >> b) & 1) ? bb : ~bb;
        }
        int lrank = popc64(peers & lanemask_lt());
#pragma unroll
        for (int q = 0; q < RS_WAVES; ++q) wcnt[q][tid] = 0;
        __syncthreads();
        if (valid && lrank == 0) wcnt[w][d] = (uint32_t)popc64(peers);
        __syncthreads();
        if (valid) {
            uint32_t before = 0;
            for (int q = 0; q < w; ++q) before += wcnt[q][d];
            int64_t pos = off[(int64_t)d * nb + blockIdx.x] + run[d] + before + lrank;
            if (kout) kout[pos] = key;
            if (vout) vout[pos] = val;
        }
        __syncthreads();
        uint32_t add = 0;
#pragma unroll
        for (int q = 0; q < RS_WAVES; ++q) add += wcnt[q][tid];
        run[tid] += add;
        __syncthreads();
    }
}

}  // namespace

int64_t scan_tmp_elems(int64_t n) { return (n + SCAN_TILE - 1) / SCAN_TILE + 1; }

hipError_t exclusive_scan_i32(const int32_t* in, int64_t* out, int64_t n, int64_t* d_total, int64_t* tmp,
                              hipStream_t s) {
    return scan_impl<int32_t>(in, out, n, d_total, tmp, s);
}
hipError_t exclusive_scan_i64(const int64_t* in, int64_t* out, int64_t n, int64_t* d_total, int64_t* tmp,
                              hipStream_t s) {
    return scan_impl<int64_t>(in, out, n, d_total, tmp, s);
}

// (of a short sort also what a longer one of up to the limit needs, so that a
// buffer sized for n serves any smaller sort)
int64_t radix_hist_elems(int64_t n, bool small_hist) {
    if (small_hist) return 256 * rs_blocks(n, true) + 1;
    return 256 * std::max(rs_blocks(n), rs_blocks(std::min(n, RS_SHORT_N))) + 1;
}
int radix_passes(int64_t n, int bits) { return n <= 1 || bits <= 0 ? 0 : (bits + 7) / 8; }

template <typename K>
static void rs_hist(const K* keys, int64_t n, int shift, int64_t* hist, hipStream_t s, bool small_hist) {
    const int64_t nb = rs_blocks(n, small_hist);
    if (rs_short(n, small_hist))
        hipLaunchKernelGGL((k_rs_hist<K, RS_ITEMS_SHORT>), dim3((unsigned)nb), dim3(RS_BLOCK), 0, s, keys, n, shift, nb,
                           hist);
    else
        hipLaunchKernelGGL((k_rs_hist<K, RS_ITEMS>), dim3((unsigned)nb), dim3(RS_BLOCK), 0, s, keys, n, shift, nb, hist);
}
template <typename K>
static void rs_scatter(const K* kin, const uint32_t* vin, K* kout, uint32_t* vout, int64_t n, int shift,
                       const int64_t* off, hipStream_t s, bool small_hist) {
    const int64_t nb = rs_blocks(n, small_hist);
    if (rs_short(n, small_hist))
        hipLaunchKernelGGL((k_rs_scatter<K, RS_ITEMS_SHORT>), dim3((unsigned)nb), dim3(RS_BLOCK), 0, s, kin, vin, kout,
                           vout, n, shift, nb, off);
    else
        hipLaunchKernelGGL((k_rs_scatter<K, RS_ITEMS>), dim3((unsigned)nb), dim3(RS_BLOCK), 0, s, kin, vin, kout, vout, n,
                           shift, nb, off);
}

hipError_t bin_sort_u8(const uint8_t* keys, int64_t n, uint32_t* out, int64_t* hist, int64_t* tmp, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    rs_hist(keys, n, 0, hist, s, false);
    hipError_t e = exclusive_scan_i64(hist, hist, 256 * rs_blocks(n), nullptr, tmp, s);
    if (e != hipSuccess) return e;
    rs_scatter(keys, nullptr, (uint8_t*)nullptr, out, n, 0, hist, s, false);
    return hipGetLastError();
}

template <typename K>
static hipError_t radix_sort(K* keys, uint32_t* vals, K* keys_alt, uint32_t* vals_alt, int64_t n, int bits,
                             int64_t* hist, int64_t* tmp, hipStream_t s, bool copy_back, bool small_hist) {
    const int passes = radix_passes(n, bits);
    K *ka = keys, *kb = keys_alt;
    uint32_t *va = vals, *vb = vals ? vals_alt : nullptr;
    for (int p = 0; p < passes; ++p) {
        rs_hist(ka, n, p * 8, hist, s, small_hist);
        hipError_t e = exclusive_scan_i64(hist, hist, 256 * rs_blocks(n, small_hist), nullptr, tmp, s);
        if (e != hipSuccess) return e;
        rs_scatter(ka, va, kb, vb, n, p * 8, hist, s, small_hist);
        K* kt = ka; ka = kb; kb = kt;
        uint32_t* vt = va; va = vb; vb = vt;
    }
    if ((passes & 1) && copy_back) {
        hipError_t e = hipMemcpyAsync(keys, ka, sizeof(K) * n, hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return e;
        if (vals) e = hipMemcpyAsync(vals, va, sizeof(uint32_t) * n, hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

hipError_t radix_sort_u64(uint64_t* keys, uint32_t* vals, uint64_t* keys_alt, uint32_t* vals_alt, int64_t n,
                          int bits, int64_t* hist, int64_t* tmp, hipStream_t s, bool small_hist) {
    return radix_sort<uint64_t>(keys, vals, keys_alt, vals_alt, n, bits, hist, tmp, s, true, small_hist);
}
hipError_t radix_sort_u32(uint32_t* keys, uint32_t* vals, uint32_t* keys_alt, uint32_t* vals_alt, int64_t n,
                          int bits, int64_t* hist, int64_t* tmp, hipStream_t s, bool copy_back) {
    return radix_sort<uint32_t>(keys, vals, keys_alt, vals_alt, n, bits, hist, tmp, s, copy_back, false);
}

}  // namespace ebb
