// count.hip -- host orchestration of counting: the sub-branch arena, task
// generation and the per-width-class search launches.
//
// Seeds.  Every k-clique is counted under the edge of the clique that comes
// first in pi_tau (Section 4.1), inside that edge's sub-branch g_i, which
// needs at least k-2 vertices.  The arena keeps g_i for every edge with
// |V(g_i)| >= 1, in rank order, so a rank range is a slot range.
//
// Tasks.  For a count at k, every slot with |V(g_i)| >= k-2 becomes one task;
// a slot whose root has more than split_threshold (k-2)-subsets becomes one
// task per possible first vertex x of the root's children.  Tasks are sorted
// by bitmap width class, and inside a class by the number of vertices the
// task's subtree can still use, largest first, so heavy work starts first.
#include <algorithm>
#include <cmath>
#include <mutex>

#include "arena.h"
#include "common.h"
#include "handle.h"
#include "prims.h"
#include "slab.h"

namespace ebb {

namespace {

std::once_flag g_binom_once[64];
hipError_t g_binom_err[64];

hipError_t ensure_binom(int dev, hipStream_t s) {
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::call_once(g_binom_once[dev], [&] {
        g_binom_err[dev] = launch_binom_init(s);
        if (g_binom_err[dev] == hipSuccess) g_binom_err[dev] = hipStreamSynchronize(s);
    });
    return g_binom_err[dev];
}

int opts_of(const ebbkc_options& o) {
    int f = 0;
    if (o.early_termination) f |= OPT_ET;
    if (o.rule1) f |= OPT_RULE1;
    if (o.rule2) f |= OPT_RULE2;
    if (o.count_work) f |= OPT_WORK;
    return f;
}

// counters: [0..4) per-class work queues, [4,5] total lo/hi, [6] error flags,
// [12..16) per-class task counts (task generation), [16 + 4 (W-1) ..) search
// work of width class W (tasks, nodes, word operations), [32 + 4 (W-1) ..)
// its waves' end times (sum, latest, count, ~earliest start), [48 + W-1]
// nodes it handed over through the split queue
constexpr int CNT_WORDS = 64;

GraphView graph_view(const ebbkc_graph* g) {
    return GraphView{g->rp, g->ci, g->erank, g->rrow, g->orp, g->orow, g->eu, g->ev, g->rank,
                     g->adj, g->acum, g->adjw};
}

__host__ __device__ inline int width_of(int c) { return c <= 64 ? 1 : (c <= 128 ? 2 : (c <= 192 ? 3 : 4)); }

inline unsigned grid_for(int64_t n, int per = 256) {
    int64_t b = (n + per - 1) / per;
    if (b < 1) b = 1;
    if (b > 16384) b = 16384;
    return (unsigned)b;
}

// ---------------------------------------------------------------- kernels

// Slots: the items (ranks, or positions of the vertex order) with a non-empty
// sub-branch, in order.  One tile of items per workgroup: k_seed_sums adds up
// its slots, vertices and row words (and the slots of every size), k_seed_parts
// turns the tile sums into offsets, k_seed_fill reads the tile again and writes
// its slots.  Inside a tile the three sums travel as one 64-bit word (at most
// 2^11 slots, 2^19 vertices, 2^21 row words), so one scan serves all three.
constexpr int SEED_BLOCK = 256, SEED_ITEMS = 8, SEED_TILE = SEED_BLOCK * SEED_ITEMS;
constexpr int SIZE_BINS = 64 * MAX_W + 1;

struct SeedSums {
    int64_t slots, vtx, words;
};

__device__ __forceinline__ int seed_size(const int32_t* __restrict__ id, const int32_t* __restrict__ size,
                                         bool by_id, int64_t r) {
    return by_id ? size[id[r]] : size[r];
}
__device__ __forceinline__ uint64_t seed_pack(int c) {
    return c > 0 ? (1ull << 48) | ((uint64_t)c << 24) | (uint64_t)(c * width_of(c)) : 0ull;
}

__global__ __launch_bounds__(SEED_BLOCK) void k_seed_sums(const int32_t* __restrict__ id,
                                                          const int32_t* __restrict__ size, bool by_id, int64_t n,
                                                          SeedSums* __restrict__ part,
                                                          unsigned long long* __restrict__ bins, int* __restrict__ err) {
    __shared__ uint32_t h[SIZE_BINS];
    __shared__ uint64_t ws[SEED_BLOCK / EBB_WAVE];
    for (int i = threadIdx.x; i < SIZE_BINS; i += SEED_BLOCK) h[i] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * SEED_TILE;
    uint64_t acc = 0;
#pragma unroll
    for (int j = 0; j < SEED_ITEMS; ++j) {
        const int64_t r = base + j * SEED_BLOCK + threadIdx.x;
        if (r >= n) continue;
        int c = seed_size(id, size, by_id, r);
        if (c <= 0) continue;
        if (c > 64 * MAX_W) {
            atomicOr(err, ERR_WIDTH);
            c = 64 * MAX_W;
        }
        atomicAdd(&h[c], 1u);
        acc += seed_pack(c);
    }
    acc = wave_sum(acc);
    if (lane_id() == 0) ws[threadIdx.x / EBB_WAVE] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < SEED_BLOCK / EBB_WAVE; ++i) acc += ws[i];
        part[blockIdx.x] = SeedSums{(int64_t)(acc >> 48), (int64_t)((acc >> 24) & 0xFFFFFF), (int64_t)(acc & 0xFFFFFF)};
    }
    for (int i = threadIdx.x; i < SIZE_BINS; i += SEED_BLOCK)
        if (h[i]) atomicAdd(&bins[i], (unsigned long long)h[i]);
}

// one workgroup: exclusive scan of the tile sums in place, the totals in *tot
__global__ __launch_bounds__(SEED_BLOCK) void k_seed_parts(SeedSums* __restrict__ part, int64_t np,
                                                           SeedSums* __restrict__ tot) {
    __shared__ SeedSums wt[SEED_BLOCK / EBB_WAVE];
    const int lane = lane_id(), w = threadIdx.x / EBB_WAVE;
    SeedSums carry{0, 0, 0};
    for (int64_t base = 0; base < np; base += SEED_BLOCK) {
        const int64_t i = base + threadIdx.x;
        const SeedSums v = i < np ? part[i] : SeedSums{0, 0, 0};
        const SeedSums inc{wave_incl_scan(v.slots), wave_incl_scan(v.vtx), wave_incl_scan(v.words)};
        if (lane == EBB_WAVE - 1) wt[w] = inc;
        __syncthreads();
        SeedSums b = carry;
        for (int q = 0; q < SEED_BLOCK / EBB_WAVE; ++q) {
            const SeedSums t = wt[q];
            if (q < w) {
                b.slots += t.slots;
                b.vtx += t.vtx;
                b.words += t.words;
            }
            carry.slots += t.slots;
            carry.vtx += t.vtx;
            carry.words += t.words;
        }
        if (i < np) part[i] = SeedSums{b.slots + inc.slots - v.slots, b.vtx + inc.vtx - v.vtx, b.words + inc.words - v.words};
        __syncthreads();
    }
    if (threadIdx.x == 0) *tot = carry;
}

// The slots of each tile: id, size, offsets, and the sort key of the slot
// order (class ascending, sizes descending: size 64 W - i of class W is bin
// 64 (W - 1) + i).  rthr (vertex slots): an item's out-edges start at the rank
// equal to the vertices of the slots before it; the threshold is one below.
// next (by rank): where launch_candidates writes a slot's members.
__global__ __launch_bounds__(SEED_BLOCK) void k_seed_fill(const int32_t* __restrict__ id,
                                                          const int32_t* __restrict__ size, bool by_id, int64_t n,
                                                          const SeedSums* __restrict__ part,
                                                          int32_t* __restrict__ seed_id, int32_t* __restrict__ seed_c,
                                                          int32_t* __restrict__ rthr, int64_t* __restrict__ row_off,
                                                          int64_t* __restrict__ vtx_off, uint8_t* __restrict__ key,
                                                          unsigned long long* __restrict__ next) {
    __shared__ uint64_t ws[SEED_BLOCK / EBB_WAVE];
    const int lane = lane_id(), w = threadIdx.x / EBB_WAVE;
    SeedSums b = part[blockIdx.x];
    const int64_t base = (int64_t)blockIdx.x * SEED_TILE;
    for (int j = 0; j < SEED_ITEMS; ++j) {
        const int64_t r = base + j * SEED_BLOCK + threadIdx.x;
        const int c = r < n ? seed_size(id, size, by_id, r) : 0;
        const uint64_t v = seed_pack(c), inc = wave_incl_scan(v);
        if (lane == EBB_WAVE - 1) ws[w] = inc;
        __syncthreads();
        uint64_t before = inc - v, all = 0;
#pragma unroll
        for (int q = 0; q < SEED_BLOCK / EBB_WAVE; ++q) {
            if (q < w) before += ws[q];
            all += ws[q];
        }
        if (c > 0) {
            const int64_t s = b.slots + (int64_t)(before >> 48), vo = b.vtx + (int64_t)((before >> 24) & 0xFFFFFF);
            seed_id[s] = id[r];
            seed_c[s] = c;
            row_off[s] = b.words + (int64_t)(before & 0xFFFFFF);
            vtx_off[s] = vo;
            if (rthr) rthr[s] = (int32_t)(vo - 1);
            if (next) next[r] = (unsigned long long)vo;
            const int W = width_of(c);
            key[s] = (uint8_t)(64 * (W - 1) + 64 * W - c);
        }
        b.slots += (int64_t)(all >> 48);
        b.vtx += (int64_t)((all >> 24) & 0xFFFFFF);
        b.words += (int64_t)(all & 0xFFFFFF);
        __syncthreads();
    }
}

__global__ void k_seed_ranks(const int32_t* __restrict__ seed_eid, const int32_t* __restrict__ rank, int64_t n,
                             int32_t* __restrict__ out) {
    for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s < n; s += (int64_t)gridDim.x * blockDim.x)
        out[s] = rank[seed_eid[s]];
}

// node-parallel roots: |N+(v)| (neighbours later in the vertex order) per vertex
__global__ void k_vertex_out(const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                             const int32_t* __restrict__ vpos, int32_t n, int32_t* __restrict__ cout,
                             int32_t* __restrict__ byvpos) {
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        const int32_t pv = vpos[v];
        int32_t c = 0;
        for (int32_t j = rp[v]; j < rp[v + 1]; ++j) c += vpos[ci[j]] > pv;
        cout[pv] = c;  // indexed by position
        byvpos[pv] = (int32_t)v;
    }
}

// Listed edges: the slot of edge eids[i] by binary search of its rank in the
// slots' ranks (ascending), as a whole-root task, and the bin that sorts the
// tasks by class, larger sub-branches first (sizes 64 W - 2 q and one less are
// bin 32 (W - 1) + q; QUERY_BINS, not counted: no task).  An id that is no edge
// sets the top bit of bins[0] (counts stay below it).  Bound by latency: a chain of
// about 2 log2(slots) loads per lane.
constexpr int QUERY_BINS = 32 * MAX_W;
constexpr unsigned int QUERY_BAD = 1u << 31;
__global__ __launch_bounds__(256) void k_query_tasks(const int64_t* __restrict__ eids, int64_t n, int64_t m, int l0,
                                                     const int32_t* __restrict__ rank,
                                                     const int32_t* __restrict__ seed_eid,
                                                     const int32_t* __restrict__ seed_c, int64_t nseeds,
                                                     int64_t* __restrict__ tasks, uint8_t* __restrict__ key,
                                                     unsigned int* __restrict__ bins) {
    __shared__ unsigned int h[QUERY_BINS];
    for (int i = threadIdx.x; i < QUERY_BINS; i += blockDim.x) h[i] = 0;
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t e = eids[i];
        int b = QUERY_BINS;
        int64_t task = 0;
        if (e < 0 || e >= m) {
            atomicOr(&bins[0], QUERY_BAD);
        } else {
            const int32_t r = rank[e];
            int64_t lo = 0, hi = nseeds;
            while (lo < hi) {
                const int64_t mid = (lo + hi) >> 1;
                if (rank[seed_eid[mid]] < r) lo = mid + 1; else hi = mid;
            }
            const int c = lo < nseeds && seed_eid[lo] == (int32_t)e ? seed_c[lo] : 0;
            if (c >= l0) {
                b = 32 * (width_of(c) - 1) + ((64 * width_of(c) - c) >> 1);
                task = task_pack(lo, 0, c);
            }
        }
        tasks[i] = task;
        key[i] = (uint8_t)b;
        if (b < QUERY_BINS) atomicAdd(&h[b], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < QUERY_BINS; i += blockDim.x)
        if (h[i]) atomicAdd(&bins[i], h[i]);
}

// results of the sorted tasks to their queries; the queries without a task 0
__global__ void k_query_results(const uint64_t* __restrict__ per_task, const uint32_t* __restrict__ idx, int64_t nt,
                                int64_t n, uint64_t* __restrict__ out) {
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x)
        out[idx[j]] = j < nt ? per_task[j] : 0;
}

// root ranges of the slots of one size: segment j is the range [x0, x1) of
// every one of the slots order[first ..]; its tasks start at pref[j]
struct TaskSeg {
    int64_t pref;
    int32_t first;
    int16_t x0, x1;
};

__global__ void k_task_expand(const TaskSeg* __restrict__ seg, int nseg, int64_t n, const int32_t* __restrict__ order,
                              int64_t* __restrict__ tasks) {
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) {
        int lo = 0, hi = nseg;  // the last segment starting at or before t
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (seg[mid].pref <= t) lo = mid; else hi = mid;
        }
        const TaskSeg g = seg[lo];
        tasks[t] = task_pack(order[g.first + (t - g.pref)], g.x0, g.x1);
    }
}

__global__ void k_task_counts(const int32_t* __restrict__ seed_c, int64_t i0, int64_t n, int l0, double log_thr,
                              int32_t* __restrict__ tcount) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int c = seed_c[i0 + i];
        tcount[i] = c >= l0 ? root_tasks(c, l0, log_thr, [](int, int) {}) : 0;
    }
}

// rest: a task's class is that of the vertices from its first one on (the
// search drops the others), else its slot's
__global__ void k_task_fill(const int32_t* __restrict__ seed_c, int64_t i0, int64_t n, int l0, double log_thr, bool rest,
                            const int64_t* __restrict__ toff, int64_t* __restrict__ tasks, uint64_t* __restrict__ keys,
                            uint32_t* __restrict__ vals, unsigned long long* __restrict__ cls_count) {
    uint64_t per_class[4] = {0, 0, 0, 0};  // tasks per width class, added once per wave below
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int c = seed_c[i0 + i];
        if (c < l0) continue;
        int64_t o = toff[i];
        root_tasks(c, l0, log_thr, [&](int x0, int x1) {
            const int W = width_of(rest ? c - x0 : c);
            tasks[o] = task_pack(i0 + i, x0, x1);
            // heaviest first: more vertices after the first one of the range
            const int usable = x0 == 0 && x1 >= c ? c : c - 1 - x0;
            keys[o] = ((uint64_t)(W - 1) << 8) | (uint64_t)(255 - (usable > 255 ? 255 : usable));
            vals[o] = (uint32_t)o;
            ++o;
#pragma unroll
            for (int w = 0; w < 4; ++w) per_class[w] += w == W - 1;
        });
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const uint64_t t = wave_sum(per_class[w]);
        if (lane_id() == 0 && t) atomicAdd(&cls_count[w], (unsigned long long)t);
    }
}

__global__ void k_gather_tasks(const int64_t* __restrict__ tasks, const uint32_t* __restrict__ idx, int64_t n,
                               int64_t* __restrict__ out) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = tasks[idx[i]];
}

// sum of a per-item value over [lo, hi): k = 3 sums |V(g_i)| by rank, k = 4 |E(g_i)| by slot
__global__ void k_sum_range(const int32_t* __restrict__ byrank, const int32_t* __restrict__ vals32,
                            const uint64_t* __restrict__ vals64, int64_t lo, int64_t hi,
                            unsigned long long* __restrict__ out) {
    uint64_t acc = 0;
    for (int64_t i = lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < hi; i += (int64_t)gridDim.x * blockDim.x)
        acc += vals32 ? (uint64_t)vals32[byrank ? byrank[i] : i] : vals64[i];
    __shared__ uint64_t sm[256 / EBB_WAVE];
    block_add(acc, sm, out);
}

// bump allocator over one scratch buffer
struct Carve {
    char* base;
    size_t used, cap;
    template <typename T>
    T* take(int64_t n) {
        const size_t bytes = ((sizeof(T) * (size_t)(n > 0 ? n : 1)) + 255) & ~(size_t)255;
        if (!base || used + bytes > cap) return nullptr;
        T* p = reinterpret_cast<T*>(base + used);
        used += bytes;
        return p;
    }
};

inline size_t rnd256(size_t b) { return (b + 255) & ~(size_t)255; }

template <typename T>
struct DBuf {
    T* p = nullptr;
    hipError_t alloc(int64_t n) { return hipMalloc((void**)&p, sizeof(T) * (size_t)(n > 0 ? n : 1)); }
    ~DBuf() { if (p) (void)hipFree(p); }
    T* release() { T* q = p; p = nullptr; return q; }
};

}  // namespace

hipError_t ensure_tables(int dev, hipStream_t s) { return ensure_binom(dev, s); }

#define CHKH(expr)                                                              \
    do {                                                                        \
        hipError_t e_ = (expr);                                                 \
        if (e_ != hipSuccess) {                                                 \
            (void)hipGetLastError();                                            \
            return e_ == hipErrorOutOfMemory ? EBBKC_E_OOM : EBBKC_E_HIP;       \
        }                                                                       \
    } while (0)

void* scratch_get(ebbkc_graph* g, size_t bytes) {
    if (bytes <= g->scratch_bytes) return g->scratch;
    if (g->scratch) (void)hipFree(g->scratch);
    g->scratch = nullptr;
    g->scratch_bytes = 0;
    const size_t nb = bytes + bytes / 4;
    if (hipMalloc(&g->scratch, nb) != hipSuccess) return nullptr;
    g->scratch_bytes = nb;
    return g->scratch;
}

ebbkc_status ensure_counters(ebbkc_graph* g) {
    if (!g->d_counters) {
        if (hipMalloc((void**)&g->d_counters, CNT_WORDS * sizeof(uint64_t)) != hipSuccess) return EBBKC_E_OOM;
        if (hipHostMalloc((void**)&g->h_counters, CNT_WORDS * sizeof(uint64_t), hipHostMallocDefault) != hipSuccess)
            return EBBKC_E_OOM;
    }
    return EBBKC_OK;
}

ebbkc_status subsize_impl(ebbkc_graph* g, hipStream_t s) {
    if (g->subsize_ready) return EBBKC_OK;
    CHKH(launch_subsize(graph_view(g), g->m, g->subsize, s));
    g->subsize_ready = true;
    return EBBKC_OK;
}

// Host copy of the rank of every slot of the edge arena (rank-range counts,
// short seed lists), made on first use.
static ebbkc_status seed_ranks(ebbkc_graph* g, hipStream_t s) {
    if ((int64_t)g->seed_rank_host.size() == g->nseeds) return EBBKC_OK;
    DBuf<int32_t> r;
    CHKH(r.alloc(g->nseeds));
    hipLaunchKernelGGL(k_seed_ranks, dim3(grid_for(g->nseeds)), dim3(256), 0, s, g->seed_eid, g->rank, g->nseeds, r.p);
    CHKH(hipGetLastError());
    std::vector<int32_t> h((size_t)g->nseeds);
    CHKH(hipMemcpyAsync(h.data(), r.p, sizeof(int32_t) * g->nseeds, hipMemcpyDeviceToHost, s));
    CHKH(hipStreamSynchronize(s));
    g->seed_rank_host.swap(h);
    return EBBKC_OK;
}

// sub-branches up to this size are drawn in chunks when they are built (each
// takes a wave a few microseconds)
constexpr int BUILD_LIGHT_C = 40;

// A set of slots and their sub-branches, built from n items: ids (edges by
// rank, or vertices by position) and sizes (by id, or by item).
struct SlotSet {
    Slab held;  // all of these
    SBuf<int32_t> seed, c, rthr, order;
    SBuf<int64_t> roff, voff;
    SBuf<uint64_t> rows, ned;
    SBuf<int32_t> gid;
    SBuf<int16_t> col;
    SizeCounts count;
    SeedSums tot{0, 0, 0};
};

static ebbkc_status build_slots(ebbkc_graph* g, const int32_t* id, const int32_t* size, bool by_id, int64_t n,
                                bool vertex, SlotSet& S, hipStream_t s) {
    int* err = (int*)(g->d_counters + 6);
    const int64_t nt = (n + SEED_TILE - 1) / SEED_TILE;
    // tile sums, then the totals and the sizes' counts (read back together)
    struct Head {
        SeedSums tot;
        unsigned long long bins[SIZE_BINS];
    } h{};
    Slab tmp;
    SBuf<SeedSums> part;
    SBuf<Head> head;
    SBuf<unsigned long long> next;
    SBuf<int32_t> trows;
    SBuf<uint8_t> key;
    SBuf<int64_t> hist, htmp;
    const int64_t hn = radix_hist_elems(n), hn_tmp = scan_tmp_elems(hn) + 64, ntr = 2 + 2 * (int64_t)g->n;
    CHKH(tmp.init(SlabSize{}
                      .add<SeedSums>(nt)
                      .add<Head>(1)
                      .add<unsigned long long>(n)
                      .add<int32_t>(ntr)
                      .add<uint8_t>(n)
                      .add<int64_t>(hn)
                      .add<int64_t>(hn_tmp)));
    CHKH(part.alloc(tmp, nt));
    CHKH(head.alloc(tmp, 1));
    CHKH(hist.alloc(tmp, hn));
    CHKH(htmp.alloc(tmp, hn_tmp));
    CHKH(key.alloc(tmp, n));
    if (!vertex) {
        CHKH(next.alloc(tmp, n));
        CHKH(trows.alloc(tmp, ntr));
    }
    CHKH(hipMemsetAsync(g->d_counters, 0, CNT_WORDS * sizeof(uint64_t), s));
    CHKH(hipMemsetAsync(head.p, 0, sizeof(Head), s));
    if (n > 0) {
        hipLaunchKernelGGL(k_seed_sums, dim3((unsigned)nt), dim3(SEED_BLOCK), 0, s, id, size, by_id, n, part.p,
                           head.p->bins, err);
        hipLaunchKernelGGL(k_seed_parts, dim3(1), dim3(SEED_BLOCK), 0, s, part.p, nt, &head.p->tot);
    }
    int herr = 0;
    CHKH(hipMemcpyAsync(&h, head.p, sizeof(Head), hipMemcpyDeviceToHost, s));
    CHKH(hipMemcpyAsync(&herr, err, sizeof(int), hipMemcpyDeviceToHost, s));
    CHKH(hipStreamSynchronize(s));
    if (herr & ERR_WIDTH) return EBBKC_E_WIDTH;
    S.tot = h.tot;
    for (int c = 0; c < SIZE_BINS; ++c) S.count.n[c] = (int64_t)h.bins[c];
    const int64_t ns = S.tot.slots;
    CHKH(S.held.init(SlabSize{}
                         .add<int32_t>(ns, vertex ? 4 : 3)
                         .add<int64_t>(ns, 3)
                         .add<uint64_t>(S.tot.words)
                         .add<int32_t>(S.tot.vtx)
                         .add<int16_t>(S.tot.vtx)));
    CHKH(S.rows.alloc(S.held, S.tot.words));
    CHKH(S.gid.alloc(S.held, S.tot.vtx));
    CHKH(S.col.alloc(S.held, S.tot.vtx));
    CHKH(S.seed.alloc(S.held, ns));
    CHKH(S.c.alloc(S.held, ns));
    if (vertex) CHKH(S.rthr.alloc(S.held, ns));
    CHKH(S.order.alloc(S.held, ns));
    CHKH(S.roff.alloc(S.held, ns));
    CHKH(S.voff.alloc(S.held, ns));
    CHKH(S.ned.alloc(S.held, ns));
    if (ns == 0) return EBBKC_OK;
    hipLaunchKernelGGL(k_seed_fill, dim3((unsigned)nt), dim3(SEED_BLOCK), 0, s, id, size, by_id, n, part.p, S.seed.p,
                       S.c.p, S.rthr.p, S.roff.p, S.voff.p, key.p, next.p);
    CHKH(hipGetLastError());
    if (!vertex) CHKH(launch_candidates(graph_view(g), g->n, next.p, S.gid.p, trows.p, s));
    // the slot order: by width class, largest sub-branches first
    CHKH(bin_sort_u8(key.p, ns, (uint32_t*)S.order.p, hist.p, htmp.p, s));
    for (int W = MAX_W; W >= 1; --W) {
        const int64_t nw = S.count.of_class(W);
        if (!nw) continue;
        BuildArgs b{};
        b.G = graph_view(g);
        b.list = S.order.p + S.count.class_start(W);
        b.n = nw;
        b.heavy = S.count.larger(BUILD_LIGHT_C, W);
        b.seed_eid = S.seed.p;
        b.seed_c = S.c.p;
        b.seed_rthr = S.rthr.p;
        b.row_off = S.roff.p;
        b.vtx_off = S.voff.p;
        b.rows = S.rows.p;
        b.gid = S.gid.p;
        b.col = S.col.p;
        b.nedges = S.ned.p;
        b.vcol = g->opt.ordering == EBBKC_ORDER_COLOR ? g->vcol : nullptr;
        b.next = (unsigned long long*)(g->d_counters + W - 1);
        b.err = err;
        CHKH(launch_build(W, b, g->cu_count, s));
    }
    CHKH(hipMemcpyAsync(&herr, err, sizeof(int), hipMemcpyDeviceToHost, s));
    CHKH(hipStreamSynchronize(s));
    if (herr & ERR_WIDTH) return EBBKC_E_WIDTH;
    return EBBKC_OK;
}

ebbkc_status arena_impl(ebbkc_graph* g, hipStream_t s) {
    if (g->arena_built) return EBBKC_OK;
    ebbkc_status st = ensure_counters(g);
    if (st) return st;
    st = subsize_impl(g, s);
    if (st) return st;
    SlotSet S;
    st = build_slots(g, g->byrank, g->subsize, true, g->m, false, S, s);
    if (st) return st;
    g->nseeds = S.tot.slots;
    g->seed_eid = S.seed.p;
    g->seed_c = S.c.p;
    g->seed_order = S.order.p;
    g->seed_sizes = S.count;
    g->row_off = S.roff.p;
    g->vtx_off = S.voff.p;
    g->arows = S.rows.p;
    g->agid = S.gid.p;
    g->acol = S.col.p;
    g->nedges = S.ned.p;
    g->arena_held = S.held.release();
    g->arena_bytes = (int64_t)(S.tot.words * 8 + S.tot.vtx * 6 + S.tot.slots * 36);
    g->device_bytes += g->arena_bytes;
    g->arena_built = true;
    return EBBKC_OK;
}

// Node-parallel VBBkC (ordering DEGEN_VERTEX_NP): one slot per vertex v with a
// non-empty N+(v) (neighbours later in the degeneracy order), its sub-branch
// G[N+(v)] built by the same kernel (the neighbourhood through edges ranked
// after v's first out-edge, all edges among it), in position order.  Edges are
// ranked lexicographically by their endpoints' positions, so the vertex whose
// slot follows R out-edges has the out-edges ranked [R, R + |N+(v)|).
static ebbkc_status vertex_arena_impl(ebbkc_graph* g, hipStream_t s) {
    VertexArena& A = g->varena;
    if (A.built) return EBBKC_OK;
    ebbkc_status st = ensure_counters(g);
    if (st) return st;
    const int32_t n = g->n;
    DBuf<int32_t> cout, byvpos;
    CHKH(cout.alloc(n));
    CHKH(byvpos.alloc(n));
    if (n)
        hipLaunchKernelGGL(k_vertex_out, dim3(grid_for(n)), dim3(256), 0, s, g->rp, g->ci, g->vpos, n, cout.p,
                           byvpos.p);
    SlotSet S;
    st = build_slots(g, byvpos.p, cout.p, false, n, true, S, s);
    if (st) return st;
    A.nseeds = S.tot.slots;
    A.seed_v = S.seed.p;
    A.seed_c = S.c.p;
    A.seed_rthr = S.rthr.p;
    A.seed_order = S.order.p;
    A.seed_sizes = S.count;
    A.row_off = S.roff.p;
    A.vtx_off = S.voff.p;
    A.rows = S.rows.p;
    A.gid = S.gid.p;
    A.col = S.col.p;
    A.nedges = S.ned.p;
    A.held = S.held.release();
    A.bytes = (int64_t)(S.tot.words * 8 + S.tot.vtx * 6 + S.tot.slots * 40);
    g->device_bytes += A.bytes;
    A.built = true;
    return EBBKC_OK;
}

// exchange the edge arena of the handle with its vertex arena
static void swap_arenas(ebbkc_graph* g) {
    VertexArena& A = g->varena;
    std::swap(g->nseeds, A.nseeds);
    std::swap(g->seed_eid, A.seed_v);
    std::swap(g->seed_c, A.seed_c);
    std::swap(g->seed_order, A.seed_order);
    std::swap(g->seed_sizes, A.seed_sizes);
    std::swap(g->row_off, A.row_off);
    std::swap(g->vtx_off, A.vtx_off);
    std::swap(g->arows, A.rows);
    std::swap(g->agid, A.gid);
    std::swap(g->acol, A.col);
    std::swap(g->nedges, A.nedges);
    std::swap(g->arena_held, A.held);
    std::swap(g->arena_built, A.built);
    g->np_active = !g->np_active;
}

// A new count starts: no class has run yet.
static void reset_last(ebbkc_graph* g) {
    for (int i = 0; i < 4; ++i) {
        g->last_ms[i] = 0.0;
        g->last_work[i] = 0;
        for (int j = 0; j < 4; ++j) g->last_work_class[i][j] = 0;
    }
    for (bool& b : g->tev_set) b = false;
}

// Adds the launches just made to the times and work figures of this count (a
// list of more than QUERY_CHUNK seeds takes several passes).
static ebbkc_status read_total(ebbkc_graph* g, uint64_t* out, hipStream_t s) {
    CHKH(hipMemcpyAsync(g->h_counters, g->d_counters, CNT_WORDS * sizeof(uint64_t), hipMemcpyDeviceToHost, s));
    CHKH(hipStreamSynchronize(s));
    for (int w = 0; w < MAX_W; ++w) {
        float ms = 0.f;
        if (g->tev_set[w] && hipEventElapsedTime(&ms, g->tev[w][0], g->tev[w][1]) == hipSuccess) g->last_ms[w] += ms;
        g->tev_set[w] = false;
    }
    const int err = (int)g->h_counters[6];
    if (err & ERR_WIDTH) return EBBKC_E_WIDTH;
    if (err & ERR_DEPTH) return EBBKC_E_K_RANGE;
    if (err & ERR_QUEUE) return EBBKC_E_HIP;
    // the exact total is 128 bits wide; the 64-bit result is an error past 2^64
    g->last_total[0] = g->h_counters[4];
    g->last_total[1] = g->h_counters[5];
    g->last_total_ovf = (err & ERR_OVERFLOW) != 0;
    if ((err & ERR_OVERFLOW) || g->h_counters[5] != 0) return EBBKC_E_OVERFLOW;
    *out = g->h_counters[4];
    for (int W = 1; W <= 4; ++W) {
        for (int i = 0; i < 3; ++i) {
            g->last_work_class[W - 1][i] += g->h_counters[16 + 4 * (W - 1) + i];
            g->last_work[i] += g->h_counters[16 + 4 * (W - 1) + i];
        }
        // wave-finish tail: latest end minus the mean end (10 ns ticks)
        const uint64_t* t = g->h_counters + 32 + 4 * (W - 1);
        if (t[2]) g->last_work_class[W - 1][3] += 10 * (t[1] - t[0] / t[2]);
        g->last_work[3] += g->h_counters[48 + W - 1];
    }
    return EBBKC_OK;
}

// Task list of slots [i0, i1) at l0 = k-2, sorted (width class, heaviest
// first) into `sorted`; class sizes into ccount.  Scratch comes from cv;
// small_hist as for radix_sort_u64.
static ebbkc_status make_tasks(ebbkc_graph* g, int64_t i0, int64_t n, int l0, double log_thr, bool rest, hipStream_t s,
                               Carve& cv, int64_t** sorted, int64_t* T_out, uint64_t ccount[4], bool small_hist = false) {
    int32_t* tcount = cv.take<int32_t>(n);
    int64_t* toff = cv.take<int64_t>(n + 1);
    int64_t* tmp = cv.take<int64_t>(scan_tmp_elems(n + 1) + 64);
    if (!tcount || !toff || !tmp) return EBBKC_E_OOM;
    hipLaunchKernelGGL(k_task_counts, dim3(grid_for(n)), dim3(256), 0, s, g->seed_c, i0, n, l0, log_thr, tcount);
    CHKH(exclusive_scan_i32(tcount, toff, n, toff + n, tmp, s));
    int64_t T = 0;
    CHKH(hipMemcpyAsync(&T, toff + n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    CHKH(hipStreamSynchronize(s));
    *T_out = T;
    if (T == 0) return EBBKC_OK;
    if (T >= ((int64_t)1 << 32)) return EBBKC_E_OOM;
    const int64_t hn = radix_hist_elems(T, small_hist);
    int64_t* tasks = cv.take<int64_t>(T);
    int64_t* tsorted = cv.take<int64_t>(T);
    uint64_t* keys = cv.take<uint64_t>(T);
    uint64_t* keys2 = cv.take<uint64_t>(T);
    uint32_t* vals = cv.take<uint32_t>(T);
    uint32_t* vals2 = cv.take<uint32_t>(T);
    int64_t* hist = cv.take<int64_t>(hn);
    int64_t* htmp = cv.take<int64_t>(scan_tmp_elems(hn) + 64);
    if (!tasks || !tsorted || !keys || !keys2 || !vals || !vals2 || !hist || !htmp) return EBBKC_E_OOM;
    unsigned long long* cls_count = (unsigned long long*)(g->d_counters + 12);
    CHKH(hipMemsetAsync(cls_count, 0, 4 * sizeof(uint64_t), s));
    hipLaunchKernelGGL(k_task_fill, dim3(grid_for(n)), dim3(256), 0, s, g->seed_c, i0, n, l0, log_thr, rest, toff,
                       tasks, keys, vals, cls_count);
    CHKH(radix_sort_u64(keys, vals, keys2, vals2, T, 10, hist, htmp, s, small_hist));
    hipLaunchKernelGGL(k_gather_tasks, dim3(grid_for(T)), dim3(256), 0, s, tasks, vals, T, tsorted);
    CHKH(hipGetLastError());
    CHKH(hipMemcpyAsync(ccount, cls_count, 4 * sizeof(uint64_t), hipMemcpyDeviceToHost, s));
    CHKH(hipStreamSynchronize(s));
    *sorted = tsorted;
    return EBBKC_OK;
}

// scratch bytes for make_tasks over n slots with at most T tasks
size_t task_bytes(int64_t n, int64_t T, bool small_hist) {
    const int64_t hn = radix_hist_elems(T, small_hist);
    return rnd256((size_t)n * 4) + rnd256((size_t)(n + 1) * 8) + rnd256((size_t)(scan_tmp_elems(n + 1) + 64) * 8) +
           4 * rnd256((size_t)T * 8) + 2 * rnd256((size_t)T * 4) + rnd256((size_t)hn * 8) +
           rnd256((size_t)(scan_tmp_elems(hn) + 64) * 8) + 4096;
}

// The tasks of one width class: explicit words, then whole roots of slots.
struct ClassTasks {
    const int64_t* tasks = nullptr;
    int64_t ntasks = 0;
    const int32_t* slots = nullptr;
    int64_t nslots = 0;
    int64_t first = 0;          // where the explicit words start in the list of all classes
    int64_t heavy = INT64_MAX;  // tasks drawn one at a time, the first ones
    int cmax = 64 * MAX_W;  // no sub-branch of the class's tasks is larger
};
struct TaskPlan {
    ClassTasks cls[MAX_W];
    // classes contiguous in one sorted list of explicit tasks
    static TaskPlan of_list(const int64_t* tsorted, const uint64_t ccount[4]) {
        TaskPlan p;
        for (int w = 0; w < MAX_W; ++w) {
            p.cls[w].tasks = tsorted;
            p.cls[w].ntasks = (int64_t)ccount[w];
            p.cls[w].cmax = 64 * (w + 1);
            tsorted += ccount[w];
        }
        return p;
    }
};

// Whether a search below roots of at most cmax vertices can hand a node over:
// a pushed node has l in 4 .. l0 - 2 (it is a child) and at most cmax - 2
// candidates, with at least `bound` l-subsets.  Otherwise the launch goes
// without the queue: its counters cost every wave several atomics on the same
// words, and clearing its items a launch.
static bool can_split(int l0, int cmax, uint64_t bound) {
    for (int l = 4; l <= l0 - 2; ++l) {
        if (cmax - 2 < l) break;
        double b = 1.0;
        for (int j = 1; j <= l; ++j) b = b * (cmax - 2 - l + j) / j;
        if (b * 1.0001 >= (double)bound) return true;
    }
    return false;
}

// One search launch per width class.  list = false: counts (per_task
// optional); list = true: tuples.  per_task and task_off run over the classes
// in order.  Their times are read once the stream has been waited for
// (read_total).
static ebbkc_status run_tasks(ebbkc_graph* g, int32_t k, const TaskPlan& plan,
                              uint64_t* per_task, const uint64_t* task_off, int32_t* out, void* gframes, bool list,
                              hipStream_t s, bool noalloc = false, SplitItem* squeue = nullptr,
                              unsigned long long* sq = nullptr) {
    // noalloc: no EBBkC-T rank slab and no timing events (the colour-ordered
    // search below the initial branch gives the same count under EBBkC-T)
    const bool truss = !list && !noalloc && g->opt.ordering == EBBKC_ORDER_TRUSS;
    if (truss) {  // EBBkC-T: depth limit and the per-wave rank matrices
        if (k > 2 * TRUSS_FRAMES + 3) return EBBKC_E_K_RANGE;
        if (!g->rho_slab) {
            hipError_t e = hipMalloc((void**)&g->rho_slab, truss_slab_bytes(g->cu_count));
            if (e != hipSuccess) {
                (void)hipGetLastError();
                g->rho_slab = nullptr;
                return e == hipErrorOutOfMemory ? EBBKC_E_OOM : EBBKC_E_HIP;
            }
        }
    }
    // listings up to k = 8 sort and hash each tuple as it is written
    unsigned long long* fused = list && k <= LIST_FUSED_K ? (unsigned long long*)(g->d_counters + 8) : nullptr;
    if (fused) CHKH(hipMemsetAsync(fused, 0, 2 * sizeof(uint64_t), s));
    int64_t off = 0;
    for (int W = 1; W <= MAX_W; ++W) {
        const ClassTasks& ct = plan.cls[W - 1];
        const int64_t nt = ct.ntasks + ct.nslots;
        g->tev_set[W - 1] = false;
        if (!nt) continue;
        const bool timed = !noalloc && !list;
        if (timed)
            for (hipEvent_t& e : g->tev[W - 1])
                if (!e) CHKH(hipEventCreate(&e));
        SearchArgs a{};
        a.A = ArenaView{g->seed_eid, g->seed_c, g->row_off, g->vtx_off, g->arows, g->agid, g->acol};
        a.tasks = ct.tasks;
        a.nexplicit = ct.ntasks;
        a.slots = ct.slots;
        a.ntasks = nt;
        a.heavy = ct.heavy;
        a.k = k;
        a.deep = k >= SEARCH_BRANCH_K;
        a.opts = opts_of(g->opt);
        a.k4_weight = k4_weight_of(g->opt.dense_k4);
        // under the vertex slots k is one above the clique size
        a.tplex = g->np_active && g->opt.t_plex == 0 ? (2 * (k - 1) <= g->tau ? 2 : 3) : g->opt.t_plex;
        a.tau = g->tau;
        a.next = (unsigned long long*)(g->d_counters + W - 1);
        a.total = (unsigned long long*)(g->d_counters + 4);
        a.work = (unsigned long long*)(g->d_counters + 16 + 4 * (W - 1));
        a.err = (int*)(g->d_counters + 6);
        a.per_task = per_task ? per_task + off : nullptr;
        a.task_off = task_off ? task_off + off : nullptr;
        a.out = out;
        a.eu = g->eu;
        a.ev = g->ev;
        a.list_checksums = fused;
        a.gframes = gframes;
        // runtime splitting: counts only (a queued node's count is not a task's own)
        const uint64_t bound = g->opt.node_split == 1   ? 0
                               : g->opt.node_split >= 2 ? (uint64_t)g->opt.node_split
                                                        : node_split_default(k - 2);
        if (squeue && !list && !truss && !per_task && g->opt.node_split != -1 && g->opt.blocks_per_cu != -1 &&
            can_split(k - 2, ct.cmax, bound)) {
            a.squeue = squeue;
            a.sq = sq;
            a.split_mode = g->opt.node_split == 1 ? SPLIT_FORCED : SPLIT_ON_DEMAND;
            a.split_bound = bound;
            CHKH(launch_sq_reset(sq, squeue, s));
        }
        if (g->opt.count_work && !list && !truss) a.wave_time = (unsigned long long*)(g->d_counters + 32 + 4 * (W - 1));
        if (timed) CHKH(hipEventRecord(g->tev[W - 1][0], s));
        if (list) {
            CHKH(launch_list(W, a, g->cu_count, s));
        } else if (truss) {
            TrussArgs t{};
            t.A = a.A;
            t.tasks = a.tasks;  // explicit tasks only
            t.ntasks = a.nexplicit;
            t.k = k;
            t.opts = a.opts;
            t.tplex = g->opt.t_plex;
            t.rp = g->rp;
            t.ci = g->ci;
            t.erank = g->erank;
            t.rho = g->rho_slab;
            t.next = a.next;
            t.total = a.total;
            t.work = a.work;
            t.err = a.err;
            t.per_task = a.per_task;
            CHKH(launch_search_truss(W, t, g->cu_count, s));
        } else {
            CHKH(launch_search(W, false, a, g->cu_count, g->opt.blocks_per_cu, s));
            if (a.squeue)
                CHKH(hipMemcpyAsync(g->d_counters + 48 + W - 1, sq + SQ_PUSHED, sizeof(uint64_t),
                                    hipMemcpyDeviceToDevice, s));
        }
        if (timed) {
            CHKH(hipEventRecord(g->tev[W - 1][1], s));
            g->tev_set[W - 1] = true;
        }
        off += nt;
    }
    return EBBKC_OK;
}

// A count's scratch: the handle's buffer, grown on demand, or (fixed != null)
// a fixed buffer of cap bytes that is never grown: a count that needs more
// returns EBBKC_E_SCRATCH, and nothing is allocated.
struct ScratchSrc {
    void* fixed = nullptr;
    size_t cap = 0;
};

static Carve carve_for(ebbkc_graph* g, const ScratchSrc& src, size_t bytes) {
    if (src.fixed) return Carve{bytes <= src.cap ? (char*)src.fixed : nullptr, 0, src.cap};
    char* p = (char*)scratch_get(g, bytes);
    return Carve{p, 0, p ? g->scratch_bytes : 0};
}

static ebbkc_status count_core(ebbkc_graph* g, int32_t k, int64_t r_begin, int64_t r_end, uint64_t* out,
                               hipStream_t s, const ScratchSrc& src);

// slots [*i0, *i1) of the seeds ranked in [r_begin, r_end)
static ebbkc_status slots_of_ranks(ebbkc_graph* g, int64_t r_begin, int64_t r_end, int64_t* i0, int64_t* i1,
                                   hipStream_t s) {
    ebbkc_status st = seed_ranks(g, s);
    if (st) return st;
    const auto& SR = g->seed_rank_host;
    *i0 = std::lower_bound(SR.begin(), SR.end(), (int32_t)std::min<int64_t>(r_begin, INT32_MAX)) - SR.begin();
    *i1 = std::lower_bound(SR.begin(), SR.end(), (int32_t)std::min<int64_t>(r_end, INT32_MAX)) - SR.begin();
    return EBBKC_OK;
}

// Whole roots with more than 2^18 l0-subsets are drawn one at a time: a wave
// tests about one subset per lane and instruction at worst, so a smaller root
// takes it some tens of microseconds at most, less than its share of the
// ticket counter (4,096 waves at 7 ns a ticket).
static bool heavy_root(int c, int l0) {
    double b = 1.0;
    for (int j = 1; j <= l0; ++j) b = b * (c - l0 + j) / j;
    return b > (double)(1 << 18);
}

// The tasks of every slot at l0: the root ranges of the sizes whose roots are
// split, heaviest first, as segments over the slot order (their number is
// returned, -1 past 2^32), and the sizes below them as whole roots, taken
// straight from the slot order.
static int64_t plan_whole(const SizeCounts& N, const int32_t* order, int l0, double log_thr, TaskPlan& plan,
                          std::vector<TaskSeg>& segs) {
    int64_t T = 0, pos = 0;  // pos: first slot of the size in the slot order
    struct Range {
        int usable, first, x0, x1;
        int64_t slots;
    };
    std::vector<Range> ranges[MAX_W];  // by the class of the vertices a range can use
    for (ClassTasks& ct : plan.cls) {
        ct.slots = nullptr;
        ct.cmax = 0;
        ct.heavy = 0;
    }
    for (int W = 1; W <= MAX_W; ++W) {
        ClassTasks& ct = plan.cls[W - 1];
        for (int c = 64 * W; c > 64 * (W - 1); --c) {
            const int64_t nc = N.n[c];
            if (nc == 0) continue;
            if (c >= l0) {
                if (root_split(c, l0, log_thr)) {
                    root_tasks(c, l0, log_thr, [&](int x0, int x1) {
                        const int w = width_of(c - x0) - 1;
                        ranges[w].push_back({x0 == 0 && x1 >= c ? c : c - 1 - x0, (int)pos, x0, x1, nc});
                        plan.cls[w].cmax = std::max(plan.cls[w].cmax, c - x0);
                    });
                } else {
                    ct.cmax = std::max(ct.cmax, c);
                    if (!ct.slots) ct.slots = order + pos;
                    ct.nslots += nc;
                    if (heavy_root(c, l0)) ct.heavy += nc;
                }
            }
            pos += nc;
        }
    }
    for (int w = 0; w < MAX_W; ++w) {
        ClassTasks& ct = plan.cls[w];
        std::vector<Range>& rs = ranges[w];
        std::stable_sort(rs.begin(), rs.end(), [](const Range& a, const Range& b) { return a.usable > b.usable; });
        ct.first = T;
        for (const Range& r : rs) {
            segs.push_back(TaskSeg{T, r.first, (int16_t)r.x0, (int16_t)r.x1});
            T += r.slots;
            ct.ntasks += r.slots;
            ct.heavy += r.slots;
        }
    }
    return T < ((int64_t)1 << 32) ? T : -1;
}

int64_t plan_ranges(const SizeCounts& N, int l0, double log_thr, int64_t first[MAX_W]) {
    TaskPlan plan;
    std::vector<TaskSeg> segs;
    const int64_t T = plan_whole(N, nullptr, l0, log_thr, plan, segs);
    for (int w = 0; w < MAX_W; ++w) first[w] = plan.cls[w].first;
    return T;
}

ebbkc_status count_impl(ebbkc_graph* g, int32_t k, int64_t r_begin, int64_t r_end, const int64_t* d_eids, int64_t ne,
                        uint64_t* d_per_seed, uint64_t* out, hipStream_t s) {
    (void)d_eids;
    (void)ne;
    (void)d_per_seed;
    return count_core(g, k, r_begin, r_end, out, s, ScratchSrc{});
}

static ebbkc_status count_core(ebbkc_graph* g, int32_t k, int64_t r_begin, int64_t r_end, uint64_t* out,
                               hipStream_t s, const ScratchSrc& src) {
    const bool noalloc = src.fixed != nullptr;
    const ebbkc_status e_space = noalloc ? EBBKC_E_SCRATCH : EBBKC_E_OOM;
    if (k < 3 || k > MAX_K) return EBBKC_E_K_RANGE;
    if (noalloc && (!g->arena_built || !g->d_counters || !g->subsize_ready)) return EBBKC_E_INVALID_ARG;
    if (!noalloc && g->opt.ordering == EBBKC_ORDER_DEGEN_VERTEX_NP && !g->np_active && r_begin <= 0 &&
        (r_end < 0 || r_end >= g->m) && k + 1 <= MAX_K) {
        // node-parallel VBBkC: one root per vertex v whose (k-1)-cliques in
        // G[N+(v)] are counted, i.e. the edge-slot search at k + 1 over the
        // vertex slots
        ebbkc_status st = vertex_arena_impl(g, s);
        if (st) return st;
        swap_arenas(g);
        st = count_core(g, k + 1, 0, -1, out, s, src);
        swap_arenas(g);
        return st;
    }
    ebbkc_status st = ensure_counters(g);  // allocated already under noalloc (checked above)
    if (st) return st;
    if (ensure_binom(g->device, s) != hipSuccess) return EBBKC_E_HIP;
    if (r_end < 0 || r_end > g->m) r_end = g->m;
    if (r_begin < 0) r_begin = 0;
    reset_last(g);
    unsigned long long* total = (unsigned long long*)(g->d_counters + 4);
    if (k == 3) {  // sum of |V(g_i)| over the seeds
        st = subsize_impl(g, s);
        if (st) return st;
        CHKH(hipMemsetAsync(g->d_counters, 0, CNT_WORDS * sizeof(uint64_t), s));
        if (r_end > r_begin)
            hipLaunchKernelGGL(k_sum_range, dim3(std::min(grid_for(r_end - r_begin), SUM_GRID)), dim3(256), 0, s, g->byrank, g->subsize,
                               (const uint64_t*)nullptr, r_begin, r_end, total);
        CHKH(hipGetLastError());
        return read_total(g, out, s);
    }
    st = arena_impl(g, s);
    if (st) return st;
    CHKH(hipMemsetAsync(g->d_counters, 0, CNT_WORDS * sizeof(uint64_t), s));
    int64_t i0 = 0, i1 = g->nseeds;
    const bool whole = r_begin == 0 && r_end == g->m;
    if (!whole) {
        st = slots_of_ranks(g, r_begin, r_end, &i0, &i1, s);
        if (st) return st;
    }
    const int64_t n = i1 - i0;
    if (k == 4) {  // sum of |E(g_i)| over the seeds
        if (n > 0)
            hipLaunchKernelGGL(k_sum_range, dim3(std::min(grid_for(n), SUM_GRID)), dim3(256), 0, s, (const int32_t*)nullptr,
                               (const int32_t*)nullptr, g->nedges, i0, i1, total);
        CHKH(hipGetLastError());
        return read_total(g, out, s);
    }
    if (n <= 0) return read_total(g, out, s);
    const int l0 = k - 2;
    // (the fixed scratch holds what it held with every class split)
    const double log_thr = split_log(g->opt, l0, !noalloc && g->opt.ordering != EBBKC_ORDER_TRUSS);

    // ---- tasks (the scratch is sized for the worst case: every slot split)
    const int64_t Tmax = n * (int64_t)(64 * MAX_W);
    const bool deep = k > SEARCH_DEEP_K;
    const size_t fbytes = deep ? search_frames_bytes(false, Tmax, g->cu_count, g->opt.blocks_per_cu) : 0;
    if (deep && !fbytes) return EBBKC_E_HIP;
    const size_t qbytes = rnd256((size_t)SQ_CAP * sizeof(SplitItem)) + rnd256(SQ_WORDS * sizeof(uint64_t));
    if (whole && !noalloc && g->opt.ordering != EBBKC_ORDER_TRUSS) {
        // every slot: the tasks follow from the slot order, so none is
        // counted, sorted or stored but the ranges of split roots
        TaskPlan plan;
        std::vector<TaskSeg> segs;
        const int64_t T = plan_whole(g->seed_sizes, g->seed_order, l0, log_thr, plan, segs);
        if (T < 0) return EBBKC_E_OOM;
        const size_t sbytes = rnd256(segs.size() * sizeof(TaskSeg));
        Carve cv = carve_for(g, src, rnd256((size_t)T * 8) + sbytes + rnd256(fbytes) + qbytes + 4096);
        if (!cv.base) return e_space;
        int64_t* tasks = cv.take<int64_t>(T);
        TaskSeg* dseg = cv.take<TaskSeg>((int64_t)segs.size());
        void* gframes = deep ? (void*)cv.take<char>((int64_t)fbytes) : nullptr;
        SplitItem* squeue = cv.take<SplitItem>(SQ_CAP);
        unsigned long long* sq = cv.take<unsigned long long>(SQ_WORDS);
        if (!tasks || !dseg || (deep && !gframes) || !squeue || !sq) return e_space;
        if (T > 0) {
            CHKH(hipMemcpyAsync(dseg, segs.data(), segs.size() * sizeof(TaskSeg), hipMemcpyHostToDevice, s));
            hipLaunchKernelGGL(k_task_expand, dim3(grid_for(T)), dim3(256), 0, s, dseg, (int)segs.size(), T,
                               g->seed_order, tasks);
            CHKH(hipGetLastError());
            for (ClassTasks& ct : plan.cls) ct.tasks = tasks + ct.first;
        }
        st = run_tasks(g, k, plan, nullptr, nullptr, nullptr, gframes, false, s, noalloc, squeue, sq);
        if (st) return st;
        return read_total(g, out, s);
    }
    // count the real number of tasks first with a small scratch, then size
    Carve cv0 = carve_for(g, src, task_bytes(n, 1));
    int32_t* tcount = cv0.take<int32_t>(n);
    int64_t* toff = cv0.take<int64_t>(n + 1);
    int64_t* tmp = cv0.take<int64_t>(scan_tmp_elems(n + 1) + 64);
    if (!tcount || !toff || !tmp) return e_space;
    hipLaunchKernelGGL(k_task_counts, dim3(grid_for(n)), dim3(256), 0, s, g->seed_c, i0, n, l0, log_thr, tcount);
    CHKH(exclusive_scan_i32(tcount, toff, n, toff + n, tmp, s));
    int64_t T = 0;
    CHKH(hipMemcpyAsync(&T, toff + n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    CHKH(hipStreamSynchronize(s));
    if (T == 0) return read_total(g, out, s);
    // (a fixed buffer too small for the short tiles' histograms may hold the long ones')
    const size_t rest = rnd256(fbytes) + qbytes;
    const bool small_hist = noalloc && task_bytes(n, T) + rest > src.cap;
    Carve cv = carve_for(g, src, task_bytes(n, T, small_hist) + rest);
    if (!cv.base) return e_space;
    int64_t* tsorted = nullptr;
    uint64_t ccount[4] = {0, 0, 0, 0};
    int64_t T2 = 0;
    st = make_tasks(g, i0, n, l0, log_thr, noalloc || g->opt.ordering != EBBKC_ORDER_TRUSS, s, cv, &tsorted, &T2, ccount,
                    small_hist);
    if (st) return st == EBBKC_E_OOM ? e_space : st;
    void* gframes = deep ? (void*)cv.take<char>((int64_t)fbytes) : nullptr;
    if (deep && !gframes) return e_space;
    SplitItem* squeue = cv.take<SplitItem>(SQ_CAP);
    unsigned long long* sq = cv.take<unsigned long long>(SQ_WORDS);
    if (!squeue || !sq) return e_space;

    // ---- search, one launch per width class
    st = run_tasks(g, k, TaskPlan::of_list(tsorted, ccount), nullptr, nullptr, nullptr, gframes, false, s, noalloc,
                   squeue, sq);
    if (st) return st;
    return read_total(g, out, s);
}

// The tasks of every slot at l0 when they are the slot order itself: no root
// split, no sub-branch of 256 vertices.
static bool plan_unsplit(const ebbkc_graph* g, int l0, double log_thr, TaskPlan& plan, int64_t* T) {
    const SizeCounts& N = g->seed_sizes;
    if (N.n[64 * MAX_W]) return false;
    for (int c = l0; c < 64 * MAX_W; ++c)
        if (N.n[c] && root_split(c, l0, log_thr)) return false;
    std::vector<TaskSeg> none;
    (void)plan_whole(N, g->seed_order, l0, log_thr, plan, none);
    *T = 0;
    for (const ClassTasks& ct : plan.cls) *T += ct.nslots;
    return true;
}

static int bits_for(uint64_t x) {
    int b = 0;
    while (b < 64 && (x >> b)) ++b;
    return b;
}

ebbkc_status list_impl(ebbkc_graph* g, int32_t k, int64_t r_begin, int64_t r_end, int32_t* d_buf, uint64_t cap,
                       uint32_t flags, uint64_t* out_written, uint64_t* out_checksums, hipStream_t s) {
    if (k < 1 || k > 64) return EBBKC_E_K_RANGE;
    ebbkc_status st = ensure_counters(g);
    if (st) return st;
    if (ensure_binom(g->device, s) != hipSuccess) return EBBKC_E_HIP;
    if (r_end < 0 || r_end > g->m) r_end = g->m;
    if (r_begin < 0 || r_begin > r_end) return EBBKC_E_INVALID_ARG;
    uint64_t N = 0;
    void* tmp_sort = nullptr;
    struct FreeOnExit { void*& p; ~FreeOnExit() { if (p) (void)hipFree(p); } } fe{tmp_sort};
    if (k <= 2) {
        if (k == 1 && (r_begin != 0 || r_end != g->m)) return EBBKC_E_INVALID_ARG;
        N = k == 1 ? (uint64_t)g->n : (uint64_t)(r_end - r_begin);
        *out_written = N;
        if (N > cap) return EBBKC_E_BUFFER_TOO_SMALL;
        if (N) CHKH(list_small(g->byrank, g->eu, g->ev, k == 1 ? 0 : r_begin, k == 1 ? g->n : r_end, k, d_buf, s));
    } else {
        st = arena_impl(g, s);
        if (st) return st;
        CHKH(hipMemsetAsync(g->d_counters, 0, CNT_WORDS * sizeof(uint64_t), s));
        int64_t i0 = 0, i1 = g->nseeds;
        const bool whole = r_begin == 0 && r_end == g->m;
        if (!whole) {
            st = slots_of_ranks(g, r_begin, r_end, &i0, &i1, s);
            if (st) return st;
        }
        const int64_t n = i1 - i0;
        if (n > 0) {
            const int l0 = k - 2;
            const double log_thr = split_log(g->opt, l0, false);
            // every slot and none split (nor of size 256, whose place among
            // the tasks of size 255 the order does not keep): the slot order
            // is the task order
            TaskPlan plan;
            int64_t T = 0;
            const bool by_order = whole && g->opt.ordering != EBBKC_ORDER_TRUSS && plan_unsplit(g, l0, log_thr, plan, &T);
            if (!by_order) {
                Carve cv0{(char*)scratch_get(g, task_bytes(n, 1)), 0, 0};
                cv0.cap = g->scratch_bytes;
                int32_t* tcount = cv0.take<int32_t>(n);
                int64_t* toff = cv0.take<int64_t>(n + 1);
                int64_t* tmp = cv0.take<int64_t>(scan_tmp_elems(n + 1) + 64);
                if (!tcount || !toff || !tmp) return EBBKC_E_OOM;
                hipLaunchKernelGGL(k_task_counts, dim3(grid_for(n)), dim3(256), 0, s, g->seed_c, i0, n, l0, log_thr,
                                   tcount);
                CHKH(exclusive_scan_i32(tcount, toff, n, toff + n, tmp, s));
                CHKH(hipMemcpyAsync(&T, toff + n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
                CHKH(hipStreamSynchronize(s));
            }
            if (T > 0) {
                // pass 1 runs the count kernel, pass 2 the listing kernel: frames
                // in device memory when either needs them
                const bool deep = k > std::min(SEARCH_DEEP_K, LIST_DEEP_K);
                size_t fbytes = 0;
                if (deep) {
                    fbytes = search_frames_bytes(false, T, g->cu_count, g->opt.blocks_per_cu);
                    if (!fbytes) return EBBKC_E_HIP;
                    fbytes = std::max(fbytes, (size_t)list_grid_waves(MAX_W, T, g->cu_count) * GLOBAL_FRAMES *
                                                  list_frame_bytes(MAX_W));
                }
                const size_t need = (by_order ? 4096 : task_bytes(n, T)) + rnd256(fbytes) + 2 * rnd256((size_t)(T + 1) * 8) +
                                    rnd256((size_t)(scan_tmp_elems(T + 1) + 64) * 8);
                if (!scratch_get(g, need)) return EBBKC_E_OOM;
                Carve cv{(char*)g->scratch, 0, g->scratch_bytes};
                if (!by_order) {
                    int64_t* tsorted = nullptr;
                    uint64_t ccount[4] = {0, 0, 0, 0};
                    int64_t T2 = 0;
                    st = make_tasks(g, i0, n, l0, log_thr, false, s, cv, &tsorted, &T2, ccount);
                    if (st) return st;
                    plan = TaskPlan::of_list(tsorted, ccount);
                }
                void* gframes = deep ? (void*)cv.take<char>((int64_t)fbytes) : nullptr;
                uint64_t* per_task = cv.take<uint64_t>(T + 1);
                uint64_t* task_off = cv.take<uint64_t>(T + 1);
                int64_t* stmp = cv.take<int64_t>(scan_tmp_elems(T + 1) + 64);
                if ((deep && !gframes) || !per_task || !task_off || !stmp) return EBBKC_E_OOM;
                // pass 1: per-task counts
                reset_last(g);
                CHKH(hipMemsetAsync(g->d_counters, 0, CNT_WORDS * sizeof(uint64_t), s));
                st = run_tasks(g, k, plan, per_task, nullptr, nullptr, gframes, false, s);
                if (st) return st;
                st = read_total(g, &N, s);
                if (st) return st;
                *out_written = N;
                if (N > cap) return EBBKC_E_BUFFER_TOO_SMALL;
                CHKH(exclusive_scan_i64((const int64_t*)per_task, (int64_t*)task_off, T, nullptr, stmp, s));
                // pass 2: tuples
                CHKH(hipMemsetAsync(g->d_counters, 0, CNT_WORDS * sizeof(uint64_t), s));
                st = run_tasks(g, k, plan, per_task, task_off, d_buf, gframes, true, s);
                if (st) return st;
                uint64_t herr = 0;
                CHKH(hipMemcpyAsync(&herr, g->d_counters + 6, sizeof(uint64_t), hipMemcpyDeviceToHost, s));
                CHKH(hipStreamSynchronize(s));
                if (herr & ERR_CAP) return EBBKC_E_HIP;
                if (herr & ERR_DEPTH) return EBBKC_E_K_RANGE;
            }
        }
        *out_written = N;
    }
    // k_list wrote sorted tuples and their checksums (buffer order) for 3 <= k <= 8
    const bool fused = k >= 3 && k <= LIST_FUSED_K;
    const bool resorted = (flags & EBBKC_LIST_SORTED) && N > 1;
    bool packed = false;
    if (N > 0) {
        if (!fused) CHKH(canon_tuples(d_buf, (int64_t)N, k, s));
        if (resorted) {
            const int bits = std::max(1, bits_for((uint64_t)(g->n > 0 ? g->n - 1 : 0)));
            const int64_t hn = radix_hist_elems((int64_t)N);
            // a tuple that fits one key is sorted as that key alone, and the
            // sorted tuples are unpacked and hashed in one pass
            packed = bits * k <= 64;
            if (packed) {
                const size_t bytes = 2 * rnd256(N * 8) + rnd256((size_t)hn * 8) +
                                     rnd256((size_t)(scan_tmp_elems(hn) + 64) * 8) + 4096;
                CHKH(hipMalloc(&tmp_sort, bytes));
                Carve cv{(char*)tmp_sort, 0, bytes};
                uint64_t* keys = cv.take<uint64_t>((int64_t)N);
                uint64_t* keys2 = cv.take<uint64_t>((int64_t)N);
                int64_t* hist = cv.take<int64_t>(hn);
                int64_t* htmp = cv.take<int64_t>(scan_tmp_elems(hn) + 64);
                if (!keys || !keys2 || !hist || !htmp) return EBBKC_E_OOM;
                if (N >= ((uint64_t)1 << 32)) return EBBKC_E_INVALID_ARG;
                CHKH(sort_packed_tuples(d_buf, (int64_t)N, k, bits, keys, keys2, hist, htmp,
                                        (unsigned long long*)(g->d_counters + 12), s));
            } else {
                const size_t bytes = 2 * rnd256(N * 8) + 2 * rnd256(N * 4) + rnd256((size_t)hn * 8) +
                                     rnd256((size_t)(scan_tmp_elems(hn) + 64) * 8) + rnd256(N * (size_t)k * 4) + 4096;
                CHKH(hipMalloc(&tmp_sort, bytes));
                Carve cv{(char*)tmp_sort, 0, bytes};
                uint64_t* keys = cv.take<uint64_t>((int64_t)N);
                uint64_t* keys2 = cv.take<uint64_t>((int64_t)N);
                uint32_t* idx = cv.take<uint32_t>((int64_t)N);
                uint32_t* idx2 = cv.take<uint32_t>((int64_t)N);
                int64_t* hist = cv.take<int64_t>(hn);
                int64_t* htmp = cv.take<int64_t>(scan_tmp_elems(hn) + 64);
                int32_t* tbuf = cv.take<int32_t>((int64_t)N * k);
                if (!keys || !keys2 || !idx || !idx2 || !hist || !htmp || !tbuf) return EBBKC_E_OOM;
                if (N >= ((uint64_t)1 << 32)) return EBBKC_E_INVALID_ARG;
                CHKH(sort_tuples(d_buf, (int64_t)N, k, bits, keys, keys2, idx, idx2, hist, htmp, tbuf, s));
            }
        }
    }
    if (out_checksums) {
        if (fused && !resorted && N > 0) {
            CHKH(hipMemcpyAsync(out_checksums, g->d_counters + 8, 2 * sizeof(uint64_t), hipMemcpyDeviceToHost, s));
        } else {
            if (!packed) CHKH(tuple_checksums(d_buf, (int64_t)N, k, (unsigned long long*)(g->d_counters + 12), s));
            CHKH(hipMemcpyAsync(out_checksums, g->d_counters + 12, 2 * sizeof(uint64_t), hipMemcpyDeviceToHost, s));
        }
    }
    CHKH(hipStreamSynchronize(s));
    return EBBKC_OK;
}

// ---------------------------------------------------------------- count without allocation
// The fixed scratch of ebbkc_count_noalloc: task lists, sort buffers and deep
// search frames of one count.  Each device holds its own copy from the load
// of the library to the end of the process; host code reaches it only through
// the address hipGetSymbolAddress returns for that device.
constexpr size_t NOALLOC_SCRATCH_BYTES = (size_t)256 << 20;
static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int NOALLOC_MAX_DEVICES = 64;
std::once_flag g_scratch_once[NOALLOC_MAX_DEVICES];
void* g_scratch_ptr[NOALLOC_MAX_DEVICES];
hipError_t g_scratch_err[NOALLOC_MAX_DEVICES];

// device address of the fixed scratch on device dev, looked up once per
// device with that device current
void* noalloc_scratch(int dev) {
    if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) return nullptr;
    std::call_once(g_scratch_once[dev], [dev] {
        int cur = 0;
        g_scratch_err[dev] = hipGetDevice(&cur);
        if (g_scratch_err[dev] != hipSuccess) return;
        if (cur != dev) g_scratch_err[dev] = hipSetDevice(dev);
        if (g_scratch_err[dev] == hipSuccess)
            g_scratch_err[dev] = hipGetSymbolAddress(&g_scratch_ptr[dev], HIP_SYMBOL(scratch));
        if (cur != dev) (void)hipSetDevice(cur);
        if (g_scratch_err[dev] != hipSuccess) {
            (void)hipGetLastError();
            g_scratch_ptr[dev] = nullptr;
        }
    });
    return g_scratch_err[dev] == hipSuccess ? g_scratch_ptr[dev] : nullptr;
}
}  // namespace

ebbkc_status count_noalloc_impl(ebbkc_graph* g, int32_t k, uint64_t* out, hipStream_t s) {
    void* p = noalloc_scratch(g->device);
    if (!p) return EBBKC_E_HIP;
    return count_core(g, k, 0, g->m, out, s, ScratchSrc{p, NOALLOC_SCRATCH_BYTES});
}

// Per-seed counts of a short list: the slots are looked up in host copies of
// the ranks and sizes.
static ebbkc_status count_few_seeds(ebbkc_graph* g, int32_t k, const int64_t* eids, int64_t ne, int32_t ptr_kind,
                                    uint64_t* out, hipStream_t s) {
    ebbkc_status st;
    std::vector<int64_t> he((size_t)ne);
    if (ptr_kind == EBBKC_PTR_DEVICE) CHKH(hipMemcpy(he.data(), eids, sizeof(int64_t) * ne, hipMemcpyDeviceToHost));
    else std::copy(eids, eids + ne, he.begin());
    if (g->seed_c_host.empty() && g->nseeds) {
        g->seed_c_host.resize((size_t)g->nseeds);
        CHKH(hipMemcpy(g->seed_c_host.data(), g->seed_c, sizeof(int32_t) * g->nseeds, hipMemcpyDeviceToHost));
    }
    if (g->rank_host.empty() && g->m) {
        g->rank_host.resize((size_t)g->m);
        CHKH(hipMemcpy(g->rank_host.data(), g->rank, sizeof(int32_t) * g->m, hipMemcpyDeviceToHost));
    }
    // tasks grouped by width class; task i -> output position
    std::vector<int64_t> tasks[MAX_W];
    std::vector<int64_t> where[MAX_W];
    std::vector<uint64_t> res((size_t)ne, 0);
    st = seed_ranks(g, s);
    if (st) return st;
    const auto& SR = g->seed_rank_host;
    for (int64_t i = 0; i < ne; ++i) {
        const int64_t e = he[(size_t)i];
        if (e < 0 || e >= g->m) return EBBKC_E_INVALID_ARG;
        const int32_t r = g->rank_host[(size_t)e];
        const int64_t slot = std::lower_bound(SR.begin(), SR.end(), r) - SR.begin();
        if (slot >= (int64_t)SR.size() || SR[(size_t)slot] != r) continue;  // empty sub-branch
        const int c = g->seed_c_host[(size_t)slot];
        if (c < k - 2) continue;
        tasks[width_of(c) - 1].push_back(task_pack(slot, 0, c));
        where[width_of(c) - 1].push_back(i);
    }
    uint64_t ccount[4];
    int64_t T = 0;
    for (int W = 0; W < MAX_W; ++W) { ccount[W] = tasks[W].size(); T += (int64_t)tasks[W].size(); }
    if (T) {
        const bool deep = k > SEARCH_DEEP_K;
        const size_t fbytes = deep ? search_frames_bytes(false, T, g->cu_count, g->opt.blocks_per_cu) : 0;
        if (deep && !fbytes) return EBBKC_E_HIP;
        if (!scratch_get(g, rnd256(T * 8) * 2 + rnd256(fbytes) + 4096)) return EBBKC_E_OOM;
        Carve cv{(char*)g->scratch, 0, g->scratch_bytes};
        int64_t* dt = cv.take<int64_t>(T);
        uint64_t* pt = cv.take<uint64_t>(T);
        void* gframes = deep ? (void*)cv.take<char>((int64_t)fbytes) : nullptr;
        if (!dt || !pt || (deep && !gframes)) return EBBKC_E_OOM;
        std::vector<int64_t> flat;
        flat.reserve((size_t)T);
        for (int W = 0; W < MAX_W; ++W) flat.insert(flat.end(), tasks[W].begin(), tasks[W].end());
        CHKH(hipMemcpyAsync(dt, flat.data(), sizeof(int64_t) * T, hipMemcpyHostToDevice, s));
        CHKH(hipMemsetAsync(g->d_counters, 0, CNT_WORDS * sizeof(uint64_t), s));
        st = run_tasks(g, k, TaskPlan::of_list(dt, ccount), pt, nullptr, nullptr, gframes, false, s);
        if (st) return st;
        uint64_t tot = 0;
        st = read_total(g, &tot, s);
        if (st) return st;
        std::vector<uint64_t> hp((size_t)T);
        CHKH(hipMemcpy(hp.data(), pt, sizeof(uint64_t) * T, hipMemcpyDeviceToHost));
        int64_t o = 0;
        for (int W = 0; W < MAX_W; ++W)
            for (size_t j = 0; j < where[W].size(); ++j) res[(size_t)where[W][j]] = hp[(size_t)o++];
    }
    if (ptr_kind == EBBKC_PTR_DEVICE) CHKH(hipMemcpy(out, res.data(), sizeof(uint64_t) * ne, hipMemcpyHostToDevice));
    else std::copy(res.begin(), res.end(), out);
    return EBBKC_OK;
}

// Per-seed counts for listed edge ids: one whole-root task per seed, looked
// up, sorted and gathered on the device (100,003 seeds at k = 6 on a
// 65,537-vertex R-MAT graph: 0.44 ms; with these steps on the host 9.1).  At
// most QUERY_CHUNK at a time, which bounds the scratch.
ebbkc_status count_seeds_impl(ebbkc_graph* g, int32_t k, const int64_t* eids, int64_t ne, int32_t ptr_kind,
                              uint64_t* out, hipStream_t s) {
    if (k < 3 || k > MAX_K) return EBBKC_E_K_RANGE;
    ebbkc_status st = ensure_counters(g);
    if (st) return st;
    if (ensure_binom(g->device, s) != hipSuccess) return EBBKC_E_HIP;
    st = arena_impl(g, s);
    if (st) return st;
    if (ne <= 0) return EBBKC_OK;
    reset_last(g);
    // On the device a list costs a dozen launches and one more wait, on the host
    // a search in the ranks for each seed.  Host / device in us at k = 6:
    //   seeds                            512      1,024    1,280    2,048
    //   R-MAT, 2^13 vertices           79/112  103/114  118/115  173/121
    //   R-MAT, 2^16 vertices          159/166  225/172  257/176  315/176
    //   Chung-Lu, 300,000 vertices     94/112  147/116  176/116  232/114
    //   G(2000, 0.01): no task at all   13/66    21/66    24/67    35/67
    // The larger graphs cross between 512 and 800 seeds, the smallest at 1,200,
    // and lists in which no seed has a task past 3,072.
    constexpr int64_t QUERY_FEW = 1024;
    if (ne <= QUERY_FEW) return count_few_seeds(g, k, eids, ne, ptr_kind, out, s);
    constexpr int64_t QUERY_CHUNK = (int64_t)1 << 22;
    const bool dev = ptr_kind == EBBKC_PTR_DEVICE;
    const int l0 = k - 2;
    const int64_t nc = std::min(ne, QUERY_CHUNK), hn = radix_hist_elems(nc);
    const bool deep = k > SEARCH_DEEP_K;
    const size_t fbytes = deep ? search_frames_bytes(false, nc, g->cu_count, g->opt.blocks_per_cu) : 0;
    if (deep && !fbytes) return EBBKC_E_HIP;
    if (!scratch_get(g, rnd256(nc * 8) * 5 + rnd256(nc) + rnd256(nc * 4) + rnd256((size_t)hn * 8) +
                            rnd256((size_t)(scan_tmp_elems(hn) + 64) * 8) + rnd256(fbytes) + 4096))
        return EBBKC_E_OOM;
    Carve cv{(char*)g->scratch, 0, g->scratch_bytes};
    int64_t* de = cv.take<int64_t>(nc);
    int64_t* tasks = cv.take<int64_t>(nc);
    int64_t* sorted = cv.take<int64_t>(nc);
    uint64_t* pt = cv.take<uint64_t>(nc);
    uint64_t* res = cv.take<uint64_t>(nc);
    uint8_t* key = cv.take<uint8_t>(nc);
    uint32_t* idx = cv.take<uint32_t>(nc);
    int64_t* hist = cv.take<int64_t>(hn);
    int64_t* htmp = cv.take<int64_t>(scan_tmp_elems(hn) + 64);
    unsigned int* bins = cv.take<unsigned int>(QUERY_BINS);
    void* gframes = deep ? (void*)cv.take<char>((int64_t)fbytes) : nullptr;
    if (!de || !tasks || !sorted || !pt || !res || !key || !idx || !hist || !htmp || !bins || (deep && !gframes))
        return EBBKC_E_OOM;
    // nothing is written to out before every chunk has been counted
    std::vector<uint64_t> kept(ne > nc ? (size_t)ne : 0);
    unsigned __int128 total = 0;
    bool any = false;
    for (int64_t i0 = 0; i0 < ne; i0 += nc) {
        const int64_t n = std::min(nc, ne - i0);
        if (dev) {  // device arrays are read and written in the null stream's order
            CHKH(hipMemcpy(de, eids + i0, sizeof(int64_t) * n, hipMemcpyDeviceToDevice));
            CHKH(hipStreamSynchronize(nullptr));
        } else {
            CHKH(hipMemcpyAsync(de, eids + i0, sizeof(int64_t) * n, hipMemcpyHostToDevice, s));
        }
        CHKH(hipMemsetAsync(bins, 0, sizeof(unsigned int) * QUERY_BINS, s));
        hipLaunchKernelGGL(k_query_tasks, dim3(grid_for(n)), dim3(256), 0, s, de, n, g->m, l0, g->rank, g->seed_eid,
                           g->seed_c, g->nseeds, tasks, key, bins);
        CHKH(hipGetLastError());
        CHKH(bin_sort_u8(key, n, idx, hist, htmp, s));
        hipLaunchKernelGGL(k_gather_tasks, dim3(grid_for(n)), dim3(256), 0, s, tasks, idx, n, sorted);
        CHKH(hipGetLastError());
        static_assert(sizeof(unsigned int) * QUERY_BINS <= sizeof(uint64_t) * CNT_WORDS, "pinned mirror");
        const unsigned int* hb = (const unsigned int*)g->h_counters;
        CHKH(hipMemcpyAsync(g->h_counters, bins, sizeof(unsigned int) * QUERY_BINS, hipMemcpyDeviceToHost, s));
        CHKH(hipStreamSynchronize(s));
        if (hb[0] & QUERY_BAD) return EBBKC_E_INVALID_ARG;
        uint64_t ccount[4] = {0, 0, 0, 0};
        int64_t heavy[4] = {0, 0, 0, 0}, T = 0;
        for (int b = 0; b < QUERY_BINS; ++b) {
            ccount[b / 32] += hb[b];
            if (heavy_root(64 * (b / 32 + 1) - 2 * (b % 32), l0)) heavy[b / 32] += hb[b];
            T += hb[b];
        }
        if (T == 0 && !dev && ne <= nc) {
            std::fill(out, out + ne, (uint64_t)0);
            return EBBKC_OK;
        }
        if (T) {
            TaskPlan plan = TaskPlan::of_list(sorted, ccount);
            for (int w = 0; w < MAX_W; ++w) plan.cls[w].heavy = heavy[w];
            CHKH(hipMemsetAsync(g->d_counters, 0, CNT_WORDS * sizeof(uint64_t), s));
            st = run_tasks(g, k, plan, pt, nullptr, nullptr, gframes, false, s);
            if (st) return st;
        }
        hipLaunchKernelGGL(k_query_results, dim3(grid_for(n)), dim3(256), 0, s, pt, idx, T, n, res);
        CHKH(hipGetLastError());
        if (T) {
            uint64_t tot = 0;
            st = read_total(g, &tot, s);
            if (st) return st;
            any = true;
            total += tot;
        } else {
            CHKH(hipStreamSynchronize(s));
        }
        if (ne > nc) CHKH(hipMemcpy(kept.data() + i0, res, sizeof(uint64_t) * n, hipMemcpyDeviceToHost));
    }
    if (any) {
        g->last_total[0] = (uint64_t)total;
        g->last_total[1] = (uint64_t)(total >> 64);
        if (g->last_total[1]) return EBBKC_E_OVERFLOW;
    }
    if (ne > nc) {
        if (dev) CHKH(hipMemcpy(out, kept.data(), sizeof(uint64_t) * ne, hipMemcpyHostToDevice));
        else std::copy(kept.begin(), kept.end(), out);
    } else if (dev) {
        CHKH(hipMemcpy(out, res, sizeof(uint64_t) * ne, hipMemcpyDeviceToDevice));
        CHKH(hipStreamSynchronize(nullptr));
    } else {
        CHKH(hipMemcpy(out, res, sizeof(uint64_t) * ne, hipMemcpyDeviceToHost));
    }
    return EBBKC_OK;
}

}  // namespace ebb
