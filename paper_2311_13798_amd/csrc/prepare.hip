// prepare.hip -- CSR intake, edge supports and the level-synchronous
// truss-based edge ordering (Section 4.2 of the paper, Eq. truss-based-edge),
// then the rank-tagged adjacency the branching kernels read.
//
// Pipeline (all on the device, one stream):
//   validate   rows strictly ascending, ids in range, no self-loops, symmetric
//   edge ids   edge (u,v), u<v, gets its rank in lexicographic order
//   triangles  degree orientation (a->b iff (deg a, a) < (deg b, b)); every
//              triangle is found once from its first oriented edge, counted
//              into the three edges' supports, then written as "the other two
//              edges" into each edge's incidence list
//   peel       level s, round r: every remaining edge with support <= s forms
//              the frontier; frontier edges get level s and rank (round, id);
//              each triangle destroyed in the round lowers each surviving edge
//              once (its lowest-id frontier edge does it); when no edge
//              qualifies s jumps to the smallest remaining support
//   adjacency  erank (rank of each CSR entry), rows re-sorted by rank
//              descending, and degree-oriented rows in the same order
#include <algorithm>
#include <atomic>

#include "arena.h"
#include "common.h"
#include "device_util.h"
#include "handle.h"
#include "prims.h"
#include "slab.h"

namespace ebb {
namespace {

constexpr int TB = 256;

inline unsigned grid_for(int64_t n, int per = TB) {
    int64_t b = (n + per - 1) / per;
    if (b < 1) b = 1;
    if (b > 65535 * 32) b = 65535 * 32;
    return (unsigned)b;
}

// row of CSR entry p (rp must be monotone; garbage otherwise, caught by validation)
__device__ __forceinline__ int32_t row_of(const int32_t* __restrict__ rp, int32_t n, int64_t p) {
    int lo = 0, hi = n;  // find largest u with rp[u] <= p
    while (hi - lo > 1) {
        const int mid = midpoint(lo, hi);
        if ((int64_t)rp[mid] <= p) lo = mid; else hi = mid;
    }
    return lo;
}

__global__ void k_validate_rows(const int32_t* __restrict__ rp, int32_t n, int64_t nnz, int* __restrict__ err) {
    for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u <= n; u += (int64_t)gridDim.x * blockDim.x) {
        if (u == 0 && rp[0] != 0) atomicOr(err, 1);
        if (u == n && (int64_t)rp[n] != nnz) atomicOr(err, 2);
        if (u < n && rp[u + 1] < rp[u]) atomicOr(err, 4);
    }
}

// Runs after k_validate_rows on the same stream and reads nothing through row
// offsets found bad there.
__global__ void k_validate_entries(const int32_t* __restrict__ rp, const int32_t* __restrict__ ci, int32_t n,
                                   int64_t nnz, int* __restrict__ err) {
    if (*(volatile int*)err & 7) return;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < nnz; p += (int64_t)gridDim.x * blockDim.x) {
        int32_t u = row_of(rp, n, p);
        int32_t v = ci[p];
        if (v < 0 || v >= n || v == u) { atomicOr(err, 8); continue; }
        if (p > rp[u] && ci[p - 1] >= v) { atomicOr(err, 16); continue; }
        int q = lower_bound_i32(ci, rp[v], rp[v + 1], u);
        if (q >= rp[v + 1] || ci[q] != u) atomicOr(err, 32);
    }
}

// ustart[u] = first entry of row u with neighbour > u; ucnt[u] = entries after it; degree max
__global__ void k_ustart(const int32_t* __restrict__ rp, const int32_t* __restrict__ ci, int32_t n,
                         int32_t* __restrict__ ustart, int32_t* __restrict__ ucnt, int* __restrict__ dmax) {
    for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < n; u += (int64_t)gridDim.x * blockDim.x) {
        int q = lower_bound_i32(ci, rp[u], rp[u + 1], (int32_t)u + 1);
        ustart[u] = q;
        ucnt[u] = rp[u + 1] - q;
        atomicMax(dmax, rp[u + 1] - rp[u]);
    }
}

__global__ void k_edge_ids(const int32_t* __restrict__ rp, const int32_t* __restrict__ ci, int32_t n, int64_t nnz,
                           const int32_t* __restrict__ ustart, const int64_t* __restrict__ eoff,
                           int32_t* __restrict__ eid, int32_t* __restrict__ src, int32_t* __restrict__ eu,
                           int32_t* __restrict__ ev) {
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < nnz; p += (int64_t)gridDim.x * blockDim.x) {
        int32_t u = row_of(rp, n, p);
        int32_t v = ci[p];
        int64_t e;
        if (v > u) {
            e = eoff[u] + (p - ustart[u]);
            eu[e] = u;
            ev[e] = v;
        } else {
            int q = lower_bound_i32(ci, ustart[v], rp[v + 1], u);
            e = eoff[v] + (q - ustart[v]);
        }
        eid[p] = (int32_t)e;
        src[p] = u;
    }
}

__device__ __forceinline__ bool oriented_before(int32_t a, int32_t da, int32_t b, int32_t db) {
    return da < db || (da == db && a < b);
}

// which CSR entries are out-entries under the degree orientation; nbr: the
// entry's neighbour (id-sorted rows) or rrow (rank-sorted rows)
__global__ void k_out_flags(const int32_t* __restrict__ rp, const int32_t* __restrict__ src,
                            const int32_t* __restrict__ ci, const int2* __restrict__ rrow, int64_t nnz,
                            int32_t* __restrict__ flag) {
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < nnz; p += (int64_t)gridDim.x * blockDim.x) {
        const int32_t a = src[p], b = rrow ? rrow[p].x : ci[p];
        flag[p] = oriented_before(a, rp[a + 1] - rp[a], b, rp[b + 1] - rp[b]);
    }
}

// The out-entries in row order at their scanned positions: (neighbour, edge
// id), or the rank-sorted entry itself; and the out-rows' offsets.  (One wave
// walking each row instead took 2.4 ms on R-MAT s18, whose longest row has
// 25,000 entries.)
__global__ void k_out_fill(const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                           const int32_t* __restrict__ eid, const int2* __restrict__ rrow, int32_t n, int64_t nnz,
                           const int32_t* __restrict__ flag, const int64_t* __restrict__ pos, int2* __restrict__ out,
                           int32_t* __restrict__ orp) {
    const int64_t step = (int64_t)gridDim.x * blockDim.x, t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t p = t0; p < nnz; p += step)
        if (flag[p]) out[pos[p]] = rrow ? rrow[p] : make_int2(ci[p], eid[p]);
    if (orp)
        for (int64_t a = t0; a <= n; a += step) orp[a] = rp[a] < nnz ? (int32_t)pos[rp[a]] : (int32_t)(nnz / 2);
}

// ---- triangles
// Triangle a->b, a->w, b->w (degree orientation) is found once, at a: out(a)
// is put into an LDS hash, and groups of 16 lanes stream out(b) of each b in
// out(a) through it.  Rows of up to TRI_WAVE_D entries take one wave, longer
// ones a workgroup (with a hash for TRI_BLOCK_D or TRI_HASH_D entries); rows
// past TRI_HASH_D (none below 4 M edges: an out-degree is at most sqrt(2 m))
// are searched in place.  On R-MAT s18 (82.8 M triangles) the passes take 5.3
// and 12.8 ms; a thread per edge with a binary search per entry and three
// atomics per triangle took 17.9 ms each.
//
// Of a triangle's three incidences the one of (a,b) is counted in a register
// and the one of (a,w) in LDS, so only the one of (b,w) needs a device
// atomic.  Pass 0 counts: sup[e] = all of them, nab / naw (by out-row position)
// those e has as (a,b) and as (a,w).  Pass 1 writes the incidence pairs: an
// edge's list holds its (a,b) pairs, then its (a,w) pairs, then its (b,w)
// pairs, whose next place is cursor[e].
constexpr int TRI_WAVE_D = 32, TRI_BLOCK_D = 512, TRI_HASH_D = 2816, TRI_GROUP = 16;

// open addressing over SLOTS slots, at most D of them taken (D < SLOTS)
template <int SLOTS, int D>
struct TriHash {
    int32_t key[SLOTS];
    int32_t cnt[D];  // (a,w) incidences by position in out(a)
    int16_t val[SLOTS];
};

__device__ __forceinline__ uint32_t tri_hash(int32_t w) { return ((uint32_t)w * 2654435761u) >> 12; }

template <int SLOTS, int D>
__device__ __forceinline__ void tri_insert(TriHash<SLOTS, D>& H, int32_t w, int i) {
    uint32_t h = tri_hash(w);
    for (;; ++h) {
        h &= SLOTS - 1;
        if (atomicCAS(&H.key[h], -1, w) == -1) break;
    }
    H.val[h] = (int16_t)i;
}

template <int SLOTS, int D>
__device__ __forceinline__ int tri_find(const TriHash<SLOTS, D>& H, int32_t w) {
    uint32_t h = tri_hash(w);
    for (;;) {
        h &= SLOTS - 1;
        const int32_t k = H.key[h];
        if (k == w) return H.val[h];
        if (k < 0) return -1;
        ++h;
    }
}

// Pass 2 runs over the rank-tagged rows (orow holds ranks instead of edge ids)
// and gives each triangle's first edge its opposite vertex: cursor by rank,
// gid the members (6.8 ms on R-MAT s18, where the search of every seed's
// shorter row prefix in the other endpoint's row was most of a small
// sub-branch's build).
struct TriArgs {
    const int32_t* orp;
    const int2* orow;
    int32_t n;
    int32_t* sup;
    int32_t* nab;
    int32_t* naw;
    const int64_t* inc_off;
    unsigned long long* cursor;
    int2* inc;
    int32_t* gid;
    const int32_t *rp, *ci, *erank;  // id-sorted rows (pass 2)
};

// The b of out(a) numbered first, first + stride, ... by a group of lanes
template <int PASS, class Find, class Count, class Rank>
__device__ __forceinline__ void tri_stream(const TriArgs& T, int a, int a0, int d, int first, int stride, Find&& find,
                                           Count&& count_aw, Rank&& rank_aw) {
    const int gl = lane_id() & (TRI_GROUP - 1), gbase = lane_id() & ~(TRI_GROUP - 1);
    for (int i = first; i < d; i += stride) {
        const int2 ab = T.orow[a0 + i];
        const int b0 = T.orp[ab.x], b1 = T.orp[ab.x + 1];
        int c = 0;
        int64_t at = 0;
        if (PASS == 1) at = T.inc_off[ab.y];
        int t = b0 + gl;
        int2 nxt = t < b1 ? T.orow[t] : make_int2(-1, 0);
        for (int base = b0; base < b1; base += TRI_GROUP) {
            const int2 bw = nxt;
            t += TRI_GROUP;
            nxt = t < b1 ? T.orow[t] : make_int2(-1, 0);
            const int j = bw.x >= 0 ? find(bw.x) : -1;
            if (PASS == 2) {
                if (j >= 0) {
                    const int32_t raw = rank_aw(j);
                    const int32_t r = ab.y < raw ? (ab.y < bw.y ? ab.y : bw.y) : (raw < bw.y ? raw : bw.y);
                    T.gid[atomicAdd(&T.cursor[r], 1ull)] = r == ab.y ? bw.x : r == raw ? ab.x : a;
                }
            } else if (PASS == 0) {
                if (j >= 0) {
                    ++c;
                    count_aw(j);
                    atomicAdd(&T.sup[bw.y], 1);
                }
            } else {
                const uint32_t hits = (uint32_t)(ballot(j >= 0) >> gbase) & ((1u << TRI_GROUP) - 1);
                if (j >= 0) {
                    const int32_t eaw = T.orow[a0 + j].y;
                    T.inc[at + __popc(hits & ((1u << gl) - 1))] = make_int2(eaw, bw.y);
                    T.inc[T.inc_off[eaw] + T.nab[a0 + j] + count_aw(j)] = make_int2(ab.y, bw.y);
                    T.inc[atomicAdd(&T.cursor[bw.y], 1ull)] = make_int2(ab.y, eaw);
                }
                at += __popc(hits);
            }
        }
        if (PASS == 0) {
#pragma unroll
            for (int o = TRI_GROUP / 2; o > 0; o >>= 1) c += __shfl_xor(c, o, TRI_GROUP);
            if (gl == 0) T.nab[a0 + i] = c;
        }
    }
}

// The rows with more than TRI_WAVE_D entries, listed in two sizes; list[0 / 1]
// hold the listed rows' numbers, then list + 2 the short ones and list + 2 + n
// the long ones.
__global__ void k_tri_rows(const int32_t* __restrict__ orp, int32_t n, int32_t* __restrict__ list) {
    for (int64_t base = (int64_t)blockIdx.x * blockDim.x; base < n; base += (int64_t)gridDim.x * blockDim.x) {
        const int64_t a = base + threadIdx.x;
        const int d = a < n ? orp[a + 1] - orp[a] : 0;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const bool mine = q == 0 ? d > TRI_WAVE_D && d <= TRI_BLOCK_D : d > TRI_BLOCK_D;
            const uint64_t mk = ballot(mine);
            if (!mk) continue;
            int at = 0;
            if (lane_id() == 0) at = atomicAdd(&list[q], popc64(mk));
            at = uniform_i32(at);
            if (mine) list[2 + (int64_t)q * n + at + popc64(mk & lanemask_lt())] = (int32_t)a;
        }
    }
}

// rows of up to TRI_WAVE_D entries: a wave each
template <int PASS>
__global__ __launch_bounds__(TB) void k_tri_wave(TriArgs T) {
    using Hash = TriHash<2 * TRI_WAVE_D, TRI_WAVE_D>;
    static_assert(2 * TRI_WAVE_D == EBB_WAVE, "a lane clears a slot");
    __shared__ Hash mem[TB / EBB_WAVE];
    Hash& H = mem[threadIdx.x / EBB_WAVE];
    const int lane = lane_id();
    const int wid = (int)((blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / EBB_WAVE);
    const int nw = (int)(gridDim.x * (int64_t)blockDim.x / EBB_WAVE);
    for (int64_t v = wid; v < T.n; v += nw) {
        const int a = (int)v;
        const int a0 = uniform_i32(T.orp[a]), d = uniform_i32(T.orp[a + 1]) - a0;
        if (d > TRI_WAVE_D) continue;
        if (d < 2) {
            if (PASS == 0 && d == 1 && lane == 0) T.nab[a0] = T.naw[a0] = 0;
            continue;
        }
        H.key[lane] = -1;
        if (lane < TRI_WAVE_D) H.cnt[lane] = 0;
        wave_sync();
        int2 own = make_int2(0, 0);
        if (lane < d) {
            own = T.orow[a0 + lane];
            tri_insert(H, own.x, lane);
        }
        wave_sync();
        tri_stream<PASS>(T, a, a0, d, lane / TRI_GROUP, EBB_WAVE / TRI_GROUP,
                         [&](int32_t w) { return tri_find(H, w); }, [&](int j) { return atomicAdd(&H.cnt[j], 1); },
                         [&](int j) { return T.orow[a0 + j].y; });
        wave_sync();
        if (PASS == 0 && lane < d) {
            T.naw[a0 + lane] = H.cnt[lane];
            const int add = H.cnt[lane] + T.nab[a0 + lane];
            if (add) atomicAdd(&T.sup[own.y], add);
        }
        wave_sync();
    }
}

// longer rows (list of *count): a workgroup each
template <int PASS, int SLOTS, int D>
__global__ __launch_bounds__(TB) void k_tri_block(TriArgs T, const int32_t* __restrict__ list,
                                                  const int32_t* __restrict__ count) {
    __shared__ TriHash<SLOTS, D> H;
    static_assert(D < SLOTS, "a free slot ends every search");
    const int rows = *count, first = threadIdx.x / TRI_GROUP, stride = TB / TRI_GROUP;
    for (int r = blockIdx.x; r < rows; r += gridDim.x) {
        const int a = list[r], a0 = T.orp[a], d = T.orp[a + 1] - a0;
        if (d <= D) {
            for (int i = threadIdx.x; i < SLOTS; i += TB) H.key[i] = -1;
            for (int i = threadIdx.x; i < d; i += TB) H.cnt[i] = 0;
            __syncthreads();
            for (int i = threadIdx.x; i < d; i += TB) tri_insert(H, T.orow[a0 + i].x, i);
            __syncthreads();
            tri_stream<PASS>(T, a, a0, d, first, stride, [&](int32_t w) { return tri_find(H, w); },
                             [&](int j) { return atomicAdd(&H.cnt[j], 1); }, [&](int j) { return T.orow[a0 + j].y; });
            __syncthreads();
            if (PASS == 0)
                for (int i = threadIdx.x; i < d; i += TB) T.naw[a0 + i] = H.cnt[i];
        } else {  // out(a) searched in device memory; (a,w) counted there too
            if (PASS != 2) {
                for (int i = threadIdx.x; i < d; i += TB) atomicExch(&T.naw[a0 + i], 0);
                __syncthreads();
            }
            // (the rank-tagged rows of pass 2 are not sorted by id: there the
            // CSR row is searched, where an edge to w found from b is an
            // out-edge of a too)
            const int32_t* ids = PASS == 2 ? T.ci : nullptr;
            const int s0 = PASS == 2 ? T.rp[a] : a0, s1 = PASS == 2 ? T.rp[a + 1] : a0 + d;
            tri_stream<PASS>(
                T, a, a0, d, first, stride,
                [&](int32_t w) {
                    int lo = s0, hi = s1;
                    while (lo < hi) {
                        const int mid = midpoint(lo, hi);
                        if ((ids ? ids[mid] : T.orow[mid].x) < w) lo = mid + 1; else hi = mid;
                    }
                    return lo < s1 && (ids ? ids[lo] : T.orow[lo].x) == w ? lo - s0 : -1;
                },
                [&](int j) { return atomicAdd(&T.naw[a0 + j], 1); }, [&](int j) { return T.erank[s0 + j]; });
            __syncthreads();
        }
        if (PASS == 0)
            for (int i = threadIdx.x; i < d; i += TB) {
                const int add = (d <= D ? H.cnt[i] : atomicAdd(&T.naw[a0 + i], 0)) + T.nab[a0 + i];
                if (add) atomicAdd(&T.sup[T.orow[a0 + i].y], add);
            }
        __syncthreads();
    }
}

// one pass over all rows (listed in rows by k_tri_rows)
template <int PASS>
hipError_t launch_tri(const TriArgs& T, const int32_t* rows, hipStream_t s) {
    const unsigned gw = (unsigned)std::min<int64_t>(2048, (T.n + 3) / 4), gb = (unsigned)std::min<int64_t>(2048, T.n);
    hipLaunchKernelGGL((k_tri_block<PASS, 4096, TRI_HASH_D>), dim3(gb), dim3(TB), 0, s, T, rows + 2 + T.n, rows + 1);
    hipLaunchKernelGGL((k_tri_block<PASS, 1024, TRI_BLOCK_D>), dim3(gb), dim3(TB), 0, s, T, rows + 2, rows);
    hipLaunchKernelGGL(k_tri_wave<PASS>, dim3(gw), dim3(TB), 0, s, T);
    return hipGetLastError();
}

// where the (b,w) incidences of every edge go
__global__ void k_tri_cursor(const int2* __restrict__ orow, const int32_t* __restrict__ nab,
                             const int32_t* __restrict__ naw, const int64_t* __restrict__ inc_off, int64_t m,
                             unsigned long long* __restrict__ cursor) {
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < m; q += (int64_t)gridDim.x * blockDim.x) {
        const int32_t e = orow[q].y;
        cursor[e] = (unsigned long long)(inc_off[e] + nab[q] + naw[q]);
    }
}

__global__ void k_iota(int32_t* __restrict__ a, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        a[i] = (int32_t)i;
}

__global__ void k_fill_i32(int32_t* __restrict__ a, int64_t n, int32_t v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        a[i] = v;
}

struct PeelState {
    int32_t minsup;
    int32_t pad;
    int64_t nf;
};

__global__ void k_peel_reset(PeelState* st) {
    st->minsup = 0x7fffffff;
    st->nf = 0;
}

__global__ void k_peel_flag(const int32_t* __restrict__ live, int64_t nlive, const int32_t* __restrict__ sup,
                            int32_t s, int32_t* __restrict__ flag, PeelState* __restrict__ st) {
    int32_t mn = 0x7fffffff;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nlive; i += (int64_t)gridDim.x * blockDim.x) {
        int32_t x = sup[live[i]];
        flag[i] = x <= s;
        mn = x < mn ? x : mn;
    }
    // one atomic per block
    __shared__ int32_t bm[TB / EBB_WAVE];
    mn = wave_min(mn);
    if (lane_id() == 0) bm[threadIdx.x / EBB_WAVE] = mn;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < TB / EBB_WAVE; ++i) mn = bm[i] < mn ? bm[i] : mn;
        mn = bm[0] < mn ? bm[0] : mn;
        if (mn < 0x7fffffff) atomicMin(&st->minsup, mn);
    }
}

__global__ void k_peel_compact(const int32_t* __restrict__ live, int64_t nlive, const int32_t* __restrict__ flag,
                               const int64_t* __restrict__ pos, int32_t* __restrict__ front,
                               int32_t* __restrict__ keep) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nlive; i += (int64_t)gridDim.x * blockDim.x) {
        int32_t e = live[i];
        if (flag[i]) front[pos[i]] = e;
        else keep[i - pos[i]] = e;
    }
}

// ---------------------------------------------------------------- truss peel
// The whole level-synchronous peel in one cooperative launch.  A round's
// frontier is the edges whose support reached the level in the round before:
// the decrement that takes an edge from level + 1 to level appends it to the
// next frontier, so a round costs its own triangles and one grid barrier, and
// the live edges are only scanned when the level changes.  An edge's round is
// stored when it is appended; positions in pi_tau follow afterwards by a
// stable sort of the rounds over the edge ids.  While a round runs, an edge
// already appended to the next one (round r + 1) still counts as present.
//
// The rounds are bound by latency: a chain of about seven dependent accesses
// and the barrier each, 1,245 of them on R-MAT s18 (27.2 ms, 21.8 us a round
// with its triangles) and some 850 on R-MAT of 49,999 vertices (9.7 ms, 11 us).  The host loop this replaces (six
// launches, a copy and a wait per round, every live edge read three times)
// took 90 and 51 ms.
//
// Words that several workgroups touch are read and written with relaxed
// device-scope atomics, which go past the compute units' vector caches and
// the L2s of the eight dies; a workgroup waits for its stores before it
// arrives at the barrier.  (Release / acquire fences there instead write back
// and drop whole caches: 14 us a barrier of 256 workgroups against 4.3 us,
// 1.7 us with 64.)  Every wait is bounded: past PEEL_WAIT_TICKS a workgroup
// sets the error word and returns, and so do the others.  That happens when
// some of the workgroups found no room beside other launches (another
// stream's, another process's) for that long; the peel then starts over with
// fewer of them (peel_attempts), in the end with one, which waits for nobody.
constexpr int PEEL_TB = 1024, PEEL_GROUP = 16;
// 64 workgroups, 128 from 2^20 edges on: more of them share a round's triangles,
// fewer make the barrier cheaper.  Preparing with 64 / 128, in ms: R-MAT of
// 0.44 M edges 10.8 / 11.3, 0.91 M 17.4 / 17.2, 1.9 M 28.0 / 26.7, 3.8 M 49.9 /
// 45.4 (256 take 2 ms more there); Chung-Lu with planted cliques, 1.5 M edges
// 9.6 / 9.8, 3.0 M 15.8 / 15.9; G(n, p) of 1.25 M edges 13.9 / 11.8, 1.8 M 81.6
// / 63.6.
constexpr int64_t PEEL_GRID = 64, PEEL_GRID_WIDE = 128, PEEL_WIDE_M = 1 << 20;
constexpr int PEEL_Q = 4096;      // appended edges collected per workgroup before they are written
// Edges with more than PEEL_SHORT triangles are listed and taken by a wave
// each, those with more than PEEL_LONG by the whole workgroup: a step of four
// triangles a lane costs about 3 us of dependent accesses, so a group takes a
// short edge in one step and a wave a long one in sixteen.
constexpr int PEEL_STEP = 4, PEEL_SHORT = PEEL_GROUP * PEEL_STEP, PEEL_LONG = 16 * 64 * PEEL_STEP;
constexpr int PEEL_LONGQ = 2048;
constexpr uint64_t PEEL_WAIT_TICKS = 2000000000ull;  // 20 s of the 100 MHz clock
constexpr uint32_t PEEL_WAIT_SPINS = 1u << 28;

struct PeelCtl {
    uint32_t arrived;   // barrier arrivals
    int32_t err;
    int32_t nf[3];      // frontier sizes: this round's, the next one's, and the one cleared meanwhile
    int32_t minsup[3];  // least support of the live edges, by scan; likewise
    int32_t tau, rounds;
};

struct PeelArgs {
    int32_t m;
    const int64_t* inc_off;
    const int2* inc;
    int32_t* sup;
    int32_t* rnd;      // -1 at the start
    int32_t* level;
    int32_t* subsize;  // triangles an edge is the first edge of in pi_tau
    int32_t* front[2];
    int32_t* live;     // per workgroup: its live edges (PEEL_TB * live_chunks entries each)
    int32_t live_chunks;
    PeelCtl* ctl;
};

struct PeelMem {
    int32_t q[PEEL_Q];
    int32_t lq[PEEL_LONGQ];
    int32_t qn, ln, lnext, base, mn, sum;
    int32_t ok;
    int32_t wcnt[PEEL_TB / EBB_WAVE];
};

// Every workgroup has arrived (generation gen, counted from 1) and its stores
// are done; false after PEEL_WAIT_TICKS or when another one gave up.
__device__ bool peel_barrier(PeelMem& M, PeelCtl* ctl, uint32_t gen) {
    wait_memory();
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t target = gen * gridDim.x;
        const uint64_t t0 = wall_clock64();
        int ok = 1;
        if (gridDim.x > 1) dev_add(&ctl->arrived, 1u);
        for (uint32_t spin = 0; gridDim.x > 1 && (int32_t)(dev_load(&ctl->arrived) - target) < 0; ++spin) {
            if (dev_load(&ctl->err) || wall_clock64() - t0 > PEEL_WAIT_TICKS || spin > PEEL_WAIT_SPINS) {
                dev_store(&ctl->err, 1);
                ok = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        M.ok = ok;
    }
    __syncthreads();
    asm volatile("" ::: "memory");
    return M.ok != 0;
}

// add edge e to the next frontier
__device__ __forceinline__ void peel_append(PeelMem& M, const PeelArgs& A, int32_t* next, int32_t* nf_next, int32_t e,
                                            int32_t round) {
    dev_store(&A.rnd[e], round);
    const int i = atomicAdd(&M.qn, 1);
    if (i < PEEL_Q) M.q[i] = e;
    else dev_store(&next[atomicAdd(nf_next, 1)], e);  // the queue is full: straight to the frontier
}

// write the collected edges to the next frontier
__device__ __forceinline__ void peel_flush(PeelMem& M, int32_t* next, int32_t* nf_next) {
    __syncthreads();
    const int n = M.qn < PEEL_Q ? M.qn : PEEL_Q;
    if (threadIdx.x == 0 && n) M.base = atomicAdd(nf_next, n);
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += PEEL_TB) dev_store(&next[M.base + i], M.q[i]);
    __syncthreads();
    if (threadIdx.x == 0) M.qn = 0;
}

// One triangle of frontier edge e (round r, level s): 1 when e is its first
// edge in pi_tau among the edges still present; then the edges that stay lose
// one support.
__device__ __forceinline__ int peel_triangle(PeelMem& M, const PeelArgs& A, int32_t* next, int32_t* nf_next, int32_t e,
                                             int2 fg, int32_t rf, int32_t rg, int32_t r, int32_t s) {
    if ((rf >= 0 && rf < r) || (rg >= 0 && rg < r)) return 0;  // destroyed in an earlier round
    if ((rf == r && fg.x < e) || (rg == r && fg.y < e)) return 0;
    if (rf != r && atomicSub(&A.sup[fg.x], 1) == s + 1) peel_append(M, A, next, nf_next, fg.x, r + 1);
    if (rg != r && atomicSub(&A.sup[fg.y], 1) == s + 1) peel_append(M, A, next, nf_next, fg.y, r + 1);
    return 1;
}

// triangles [t, t1) of edge e, every stride-th, PEEL_STEP at a time
__device__ __forceinline__ int peel_edge(PeelMem& M, const PeelArgs& A, int32_t* next, int32_t* nf_next, int32_t e,
                                         int64_t t, int64_t t1, int stride, int32_t r, int32_t s) {
    int c = 0;
    for (; t < t1; t += PEEL_STEP * stride) {
        int2 fg[PEEL_STEP];
        int32_t rf[PEEL_STEP], rg[PEEL_STEP];
#pragma unroll
        for (int j = 0; j < PEEL_STEP; ++j) fg[j] = t + j * stride < t1 ? A.inc[t + j * stride] : make_int2(-1, -1);
#pragma unroll
        for (int j = 0; j < PEEL_STEP; ++j) {
            rf[j] = fg[j].x >= 0 ? dev_load(&A.rnd[fg[j].x]) : 0;
            rg[j] = fg[j].x >= 0 ? dev_load(&A.rnd[fg[j].y]) : 0;
        }
#pragma unroll
        for (int j = 0; j < PEEL_STEP; ++j)
            if (fg[j].x >= 0) c += peel_triangle(M, A, next, nf_next, e, fg[j], rf[j], rg[j], r, s);
    }
    return c;
}

__global__ __launch_bounds__(PEEL_TB) void k_peel(PeelArgs A) {
    __shared__ PeelMem M;
    PeelCtl* ctl = A.ctl;
    const int lane = lane_id(), wave = threadIdx.x / EBB_WAVE;
    int32_t* live = A.live + (int64_t)blockIdx.x * A.live_chunks * PEEL_TB;
    if (threadIdx.x == 0) M.qn = 0;
    __syncthreads();
    uint32_t gen = 0;
    int cur = 0;      // ctl->nf slot of the frontier in work
    int scan = 0;     // ctl->minsup slot of the next scan
    int nlive = -1;   // -1: every edge of this workgroup's chunks (chunk i of PEEL_TB edges goes to
                      // workgroup i mod grid)
    int32_t r = 0, s = 0, tau = 0;
    for (;;) {
        // ---- the live edges: those at or below s form round r's frontier,
        // the others stay listed and give the least support left
        {
            const int nxt = (cur + 1) % 3;
            int32_t* next = A.front[r & 1];
            int32_t* nf_next = &ctl->nf[nxt];
            if (blockIdx.x == 0 && threadIdx.x == 0) {
                dev_store(&ctl->nf[(cur + 2) % 3], 0);
                dev_store(&ctl->minsup[(scan + 1) % 3], 0x7fffffff);
            }
            if (threadIdx.x == 0) M.mn = 0x7fffffff;
            __syncthreads();
            const bool all = nlive < 0;
            const int total = all ? A.live_chunks * PEEL_TB : nlive;
            int kept = 0, mn = 0x7fffffff;
            for (int i0 = 0; i0 < total; i0 += PEEL_TB) {
                const int i = i0 + threadIdx.x;
                int64_t e = -1;
                if (i < total) {
                    e = all ? ((int64_t)(i0 / PEEL_TB) * gridDim.x + blockIdx.x) * PEEL_TB + threadIdx.x : live[i];
                    if (e >= A.m) e = -1;
                }
                bool keep = false;
                if (e >= 0 && dev_load(&A.rnd[e]) < 0) {
                    const int32_t x = dev_load(&A.sup[e]);
                    keep = x > s;
                    if (keep) mn = x < mn ? x : mn;
                    else peel_append(M, A, next, nf_next, (int32_t)e, r);
                }
                const uint64_t mk = ballot(keep);
                if (lane == 0) M.wcnt[wave] = popc64(mk);
                __syncthreads();  // also: every entry of the chunk is read before its place is written
                int before = 0, chunk = 0;
                for (int w = 0; w < PEEL_TB / EBB_WAVE; ++w) {
                    const int c = M.wcnt[w];
                    before += w < wave ? c : 0;
                    chunk += c;
                }
                if (keep) live[kept + before + popc64(mk & lanemask_lt())] = (int32_t)e;
                kept += chunk;
                __syncthreads();
            }
            nlive = kept;
            mn = wave_min(mn);
            if (lane == 0 && mn < 0x7fffffff) atomicMin(&M.mn, mn);
            peel_flush(M, next, nf_next);
            if (threadIdx.x == 0 && M.mn < 0x7fffffff) atomicMin(&ctl->minsup[scan], M.mn);
            if (!peel_barrier(M, ctl, ++gen)) return;
            cur = nxt;
            const int32_t least = dev_load(&ctl->minsup[scan]);
            scan = (scan + 1) % 3;
            if (dev_load(&ctl->nf[cur]) == 0) {
                if (least == 0x7fffffff) break;  // no edge is left
                s = least;
                continue;
            }
        }
        // ---- rounds at level s until no edge qualifies
        for (int nf = dev_load(&ctl->nf[cur]); nf > 0; ++r) {
            tau = s;
            const int nxt = (cur + 1) % 3;
            const int32_t* front = A.front[r & 1];
            int32_t* next = A.front[(r + 1) & 1];
            int32_t* nf_next = &ctl->nf[nxt];
            if (blockIdx.x == 0 && threadIdx.x == 0) dev_store(&ctl->nf[(cur + 2) % 3], 0);
            if (threadIdx.x == 0) M.ln = M.lnext = 0;
            __syncthreads();
            const int gl = threadIdx.x % PEEL_GROUP, g = threadIdx.x / PEEL_GROUP;
            constexpr int GROUPS = PEEL_TB / PEEL_GROUP;
            // groups of 16 lanes take an edge each, consecutive ones on different workgroups
            for (int i = g * gridDim.x + blockIdx.x; i < nf; i += GROUPS * gridDim.x) {
                const int32_t e = dev_load(&front[i]);
                const int64_t t0 = A.inc_off[e], t1 = A.inc_off[e + 1];
                if (gl == 0) A.level[e] = s;
                if (t1 - t0 > PEEL_SHORT) {
                    int at = PEEL_LONGQ;
                    if (gl == 0) at = atomicAdd(&M.ln, 1);
                    at = __shfl(at, 0, PEEL_GROUP);
                    if (at < PEEL_LONGQ) {
                        if (gl == 0) M.lq[at] = e;
                        continue;
                    }
                }
                int c = peel_edge(M, A, next, nf_next, e, t0 + gl, t1, PEEL_GROUP, r, s);
#pragma unroll
                for (int o = PEEL_GROUP / 2; o > 0; o >>= 1) c += __shfl_xor(c, o, PEEL_GROUP);
                if (gl == 0) A.subsize[e] = c;
            }
            __syncthreads();
            // the listed edges: each wave takes the next one
            const int nl = M.ln < PEEL_LONGQ ? M.ln : PEEL_LONGQ;
            bool longer = false;
            for (;;) {
                int i = 0;
                if (lane == 0) i = atomicAdd(&M.lnext, 1);
                i = uniform_i32(i);
                if (i >= nl) break;
                const int32_t e = M.lq[i];
                const int64_t t0 = A.inc_off[e], t1 = A.inc_off[e + 1];
                if (t1 - t0 > PEEL_LONG) {
                    longer = true;
                    continue;
                }
                const int c = wave_sum(peel_edge(M, A, next, nf_next, e, t0 + lane, t1, EBB_WAVE, r, s));
                if (lane == 0) A.subsize[e] = c;
            }
            // the longest ones: the whole workgroup, one after the other
            if (__syncthreads_or(longer)) {
                for (int i = 0; i < nl; ++i) {
                    const int32_t e = M.lq[i];
                    const int64_t t0 = A.inc_off[e], t1 = A.inc_off[e + 1];
                    if (t1 - t0 <= PEEL_LONG) continue;
                    if (threadIdx.x == 0) M.sum = 0;
                    __syncthreads();
                    const int c = wave_sum(peel_edge(M, A, next, nf_next, e, t0 + threadIdx.x, t1, PEEL_TB, r, s));
                    if (lane == 0 && c) atomicAdd(&M.sum, c);
                    __syncthreads();
                    if (threadIdx.x == 0) A.subsize[e] = M.sum;
                }
            }
            peel_flush(M, next, nf_next);
            if (!peel_barrier(M, ctl, ++gen)) return;
            cur = nxt;
            nf = dev_load(&ctl->nf[cur]);
        }
        s = tau + 1;  // the next level that may hold an edge
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        ctl->tau = tau;
        ctl->rounds = r;
    }
}

// Workgroups of k_peel the current device holds at once, asked for once per
// device; 0 when it cannot say.
int64_t peel_resident(int dev, int cus) {
    static std::atomic<int> known[64];
    const bool slot = dev >= 0 && dev < 64;
    int occ = slot ? known[dev].load(std::memory_order_acquire) : 0;
    if (occ == 0) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_peel, PEEL_TB, 0) != hipSuccess) {
            (void)hipGetLastError();
            return 0;
        }
        if (slot) known[dev].store(occ, std::memory_order_release);
    }
    return (int64_t)occ * cus;
}

// frontier sizes and minima before the launch
__global__ void k_peel_begin(PeelCtl* ctl, int32_t* __restrict__ rnd, int32_t m) {
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) {
        *ctl = PeelCtl{};
        for (int32_t& x : ctl->minsup) x = 0x7fffffff;
    }
    for (int32_t j = i; j < m; j += gridDim.x * blockDim.x) rnd[j] = -1;
}

__global__ void k_erank(const int32_t* __restrict__ eid, const int32_t* __restrict__ rank, int64_t nnz,
                        int32_t* __restrict__ erank) {
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < nnz; p += (int64_t)gridDim.x * blockDim.x)
        erank[p] = rank[eid[p]];
}

// The 2 m (vertex, neighbour) entries by descending rank of their edge: entry
// 2 i + h is the h-th direction of the edge of rank m - 1 - i.  A stable sort
// by vertex then gives every row its entries by descending rank.
__global__ void k_rrow_keys(const int32_t* __restrict__ byrank, const int32_t* __restrict__ eu,
                            const int32_t* __restrict__ ev, int64_t m, uint32_t* __restrict__ keys,
                            uint32_t* __restrict__ vals) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t e = byrank[m - 1 - i];
        keys[2 * i] = (uint32_t)eu[e];
        keys[2 * i + 1] = (uint32_t)ev[e];
        vals[2 * i] = (uint32_t)(2 * i);
        vals[2 * i + 1] = (uint32_t)(2 * i + 1);
    }
}

__global__ void k_gather_rrow(const uint32_t* __restrict__ perm, const int32_t* __restrict__ byrank,
                              const int32_t* __restrict__ eu, const int32_t* __restrict__ ev, int64_t m,
                              int2* __restrict__ rrow) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < 2 * m; i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t v = perm[i];
        const int32_t r = (int32_t)(m - 1 - (v >> 1)), e = byrank[r];
        rrow[i] = make_int2((v & 1) ? eu[e] : ev[e], r);
    }
}

__global__ void k_round_keys(const int32_t* __restrict__ rnd, int64_t m, uint32_t* __restrict__ keys,
                             uint32_t* __restrict__ vals) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += (int64_t)gridDim.x * blockDim.x) {
        keys[e] = (uint32_t)rnd[e];
        vals[e] = (uint32_t)e;
    }
}

// adjacency bitmap: one bit per CSR entry (a row's entries may share a word)
__global__ void k_adj_fill(const int32_t* __restrict__ src, const int32_t* __restrict__ ci, int64_t nnz, int32_t aw,
                           uint64_t* __restrict__ adj) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nnz; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t w = ci[i];
        atomicOr((unsigned long long*)&adj[(int64_t)src[i] * aw + (w >> 6)], 1ull << (w & 63));
    }
}

// acum[x aw + q] = entries of x's id-sorted row below vertex 64 q
__global__ void k_adj_cum(const int32_t* __restrict__ rp, const int32_t* __restrict__ ci, int32_t n, int32_t aw,
                          uint16_t* __restrict__ acum) {
    const int64_t total = (int64_t)n * aw;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
        const int32_t x = (int32_t)(t / aw), q = (int32_t)(t % aw);
        int lo = rp[x], hi = rp[x + 1];
        const int base = lo;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (ci[mid] < 64 * q) lo = mid + 1; else hi = mid;
        }
        acum[t] = (uint16_t)(lo - base);
    }
}

// ---- vertex orders for the root edge order of the ablation orderings

// Greedy colouring in the visiting order (degree desc, id asc), one wave per
// vertex: a vertex takes the least colour >= 1 not held by its neighbours
// earlier in that order once all of them are coloured, which is the colour
// the sequential greedy pass gives it (Jones-Plassmann rounds).  A vertex
// still waiting adds one to *pending.
constexpr int CWIN = 4096;  // colours tested per window

__device__ __forceinline__ bool visits_before(int32_t w, int32_t dw, int32_t v, int32_t dv) {
    return dw > dv || (dw == dv && w < v);
}

__global__ __launch_bounds__(TB) void k_colour_round(const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                                                     int32_t n, int32_t* col, int32_t* __restrict__ pending) {
    __shared__ uint32_t used[TB / EBB_WAVE][CWIN / 32];
    const int lane = lane_id(), wv = threadIdx.x / EBB_WAVE;
    const int64_t wid = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / EBB_WAVE;
    const int64_t nw = (int64_t)gridDim.x * blockDim.x / EBB_WAVE;
    const volatile int32_t* vcol = col;
    int waiting = 0;
    for (int64_t vv = wid; vv < n; vv += nw) {
        const int32_t v = (int32_t)vv;
        if (__builtin_amdgcn_readfirstlane(vcol[v]) != 0) continue;
        const int32_t b = rp[v], e = rp[v + 1], dv = e - b;
        bool wait = false;
        for (int32_t j = b + lane; j < e; j += EBB_WAVE) {
            const int32_t w = ci[j];
            if (visits_before(w, rp[w + 1] - rp[w], v, dv) && vcol[w] == 0) wait = true;
        }
        if (ballot(wait)) { ++waiting; continue; }
        // the least colour absent from the earlier neighbours (at most dv of them)
        for (int32_t base = 1;; base += CWIN) {
            for (int i = lane; i < CWIN / 32; i += EBB_WAVE) used[wv][i] = 0;
            wave_sync();
            for (int32_t j = b + lane; j < e; j += EBB_WAVE) {
                const int32_t w = ci[j];
                if (!visits_before(w, rp[w + 1] - rp[w], v, dv)) continue;
                const int32_t cw = vcol[w] - base;
                if (cw >= 0 && cw < CWIN) atomicOr(&used[wv][cw >> 5], 1u << (cw & 31));
            }
            wave_sync();
            int first = CWIN;
            for (int i = lane; i < CWIN / 32; i += EBB_WAVE) {
                const uint32_t f = ~used[wv][i];
                if (f) { first = i * 32 + __builtin_ctz(f); break; }
            }
            first = wave_min(first);
            wave_sync();
            if (first < CWIN) {
                if (lane == 0) col[v] = base + first;
                break;
            }
        }
    }
    if (lane == 0 && waiting) atomicAdd(pending, waiting);
}

// colour order: key (colour desc), vertex id as the value; a stable sort keeps ids ascending
__global__ void k_colour_keys(const int32_t* __restrict__ col, int32_t n, uint64_t* __restrict__ keys,
                              uint32_t* __restrict__ vals) {
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x) {
        keys[v] = (uint64_t)(0x7fffffff - col[v]);
        vals[v] = (uint32_t)v;
    }
}

__global__ void k_scatter_pos(const uint32_t* __restrict__ vals, int64_t n, int32_t* __restrict__ pos) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        pos[vals[i]] = (int32_t)i;
}

__global__ void k_degrees(const int32_t* __restrict__ rp, int32_t n, int32_t* __restrict__ deg) {
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x)
        deg[v] = rp[v + 1] - rp[v];
}

__global__ void k_core_assign(const int32_t* __restrict__ front, int64_t nf, int64_t placed, int32_t r,
                              int32_t* __restrict__ pos, int32_t* __restrict__ rnd) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nf; i += (int64_t)gridDim.x * blockDim.x) {
        pos[front[i]] = (int32_t)(placed + i);
        rnd[front[i]] = r;
    }
}

// one wave per removed vertex: its neighbours still present lose one degree
__global__ void k_core_remove(const int32_t* __restrict__ front, int64_t nf, const int32_t* __restrict__ rp,
                              const int32_t* __restrict__ ci, const int32_t* __restrict__ rnd,
                              int32_t* __restrict__ deg) {
    const int64_t wid = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / EBB_WAVE;
    const int64_t nw = (int64_t)gridDim.x * blockDim.x / EBB_WAVE;
    for (int64_t i = wid; i < nf; i += nw) {
        const int32_t v = front[i];
        for (int32_t j = rp[v] + lane_id(); j < rp[v + 1]; j += EBB_WAVE) {
            const int32_t w = ci[j];
            if (rnd[w] < 0) atomicSub(&deg[w], 1);
        }
    }
}

// edge e = (u, v): key (min pos, max pos), lexicographic
__global__ void k_lex_edge_keys(const int32_t* __restrict__ eu, const int32_t* __restrict__ ev,
                                const int32_t* __restrict__ pos, int64_t m, int32_t n, uint64_t* __restrict__ keys,
                                uint32_t* __restrict__ vals) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += (int64_t)gridDim.x * blockDim.x) {
        const int32_t a = pos[eu[e]], b = pos[ev[e]];
        keys[e] = (uint64_t)(a < b ? a : b) * (uint64_t)n + (uint64_t)(a < b ? b : a);
        vals[e] = (uint32_t)e;
    }
}

template <typename T>
struct DBuf {
    T* p = nullptr;
    hipError_t alloc(int64_t n) { return hipMalloc((void**)&p, sizeof(T) * (size_t)(n > 0 ? n : 1)); }
    ~DBuf() { if (p) (void)hipFree(p); }
    T* release() { T* q = p; p = nullptr; return q; }
};

int bits_for(uint64_t x) {
    int b = 0;
    while (b < 64 && (x >> b)) ++b;
    return b;
}

}  // namespace

hipError_t launch_candidates(const GraphView& G, int32_t n, unsigned long long* next, int32_t* gid, int32_t* rows_tmp,
                             hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipError_t e = hipMemsetAsync(rows_tmp, 0, 2 * sizeof(int32_t), s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_tri_rows, dim3(grid_for(n)), dim3(TB), 0, s, G.orp, n, rows_tmp);
    TriArgs T{};
    T.orp = G.orp;
    T.orow = G.orow;
    T.n = n;
    T.cursor = next;
    T.gid = gid;
    T.rp = G.rp;
    T.ci = G.ci;
    T.erank = G.erank;
    return launch_tri<2>(T, rows_tmp, s);
}

// Workgroups of the peel of m edges on a device that holds `resident` of them
// at once: every one of them has to run for a barrier to pass.
int64_t peel_grid(int64_t m, int64_t resident) {
    const int64_t chunks = (m + PEEL_TB - 1) / PEEL_TB;
    const int64_t want = std::min<int64_t>(m >= PEEL_WIDE_M ? PEEL_GRID_WIDE : PEEL_GRID, (chunks + 1) / 2);
    return std::max<int64_t>(1, std::min(want, resident));
}

int peel_attempts(int64_t grid, int (*attempt)(void*, int64_t), void* arg) {
    for (;; grid /= 4) {
        if (grid < 1) grid = 1;
        const int st = attempt(arg, grid);
        if (st != PEEL_AGAIN) return st;
        if (grid == 1) return EBBKC_E_HIP;
    }
}

static int64_t scan_elems(int32_t n, int64_t nnz) { return scan_tmp_elems(nnz + n + 2) + 1024; }
static int64_t peel_live_elems(int64_t nnz) { return nnz / 2 + PEEL_TB * (PEEL_GRID_WIDE + 1); }

// Slabs of the arrays the handle keeps and of the ones only prepare uses (m =
// nnz / 2 edges, if the input turns out valid): 68 and 116 bytes an edge, and
// the triangle incidence beside them.
void prepare_sizes(int32_t n, int64_t nnz, SlabSize out[2]) {
    const int64_t mm = nnz / 2, rsort = radix_hist_elems(nnz);
    out[0] = SlabSize{}
                  .add<int32_t>((int64_t)n + 1, 2)
                  .add<int32_t>(nnz, 2)
                  .add<int32_t>(mm, 7)
                  .add<int2>(nnz)
                  .add<int2>(mm);
    out[1] = SlabSize{}
                  .add<int32_t>(n, 2)
                  .add<int64_t>((int64_t)n + 1)
                  .add<int32_t>(2 + 2 * (int64_t)n)
                  .add<int64_t>(scan_elems(n, nnz))
                  .add<int32_t>(nnz, 3)
                  .add<int64_t>(nnz)
                  .add<int2>(mm)
                  .add<int32_t>(mm, 4)
                  .add<int64_t>(mm + 1, 2)
                  .add<uint32_t>(nnz, 4)
                  .add<int64_t>(rsort)
                  .add<int64_t>(scan_tmp_elems(rsort) + 64)
                  .add<PeelCtl>(1)
                  .add<int32_t>(peel_live_elems(nnz));
}

#define CHK(expr)                                   \
    do {                                            \
        hipError_t e_ = (expr);                     \
        if (e_ != hipSuccess) {                     \
            (void)hipGetLastError();                \
            return e_ == hipErrorOutOfMemory ? EBBKC_E_OOM : EBBKC_E_HIP; \
        }                                           \
    } while (0)

ebbkc_status prepare_impl(ebbkc_graph* g, const int32_t* row_ptr, const int32_t* col_idx, int32_t ptr_kind,
                          hipStream_t s) {
    const int32_t n = g->n;
    const int64_t nnz = g->nnz;
    hipEvent_t ev0, ev1;
    CHK(hipEventCreate(&ev0));
    CHK(hipEventCreate(&ev1));
    CHK(hipEventRecord(ev0, s));

    Slab held, tmp;
    SlabSize size[2];
    prepare_sizes(n, nnz, size);
    CHK(held.init(size[0]));
    CHK(tmp.init(size[1]));
    const int64_t tmp_elems = scan_elems(n, nnz), rtmp_elems = scan_tmp_elems(radix_hist_elems(nnz)) + 64;
    const int64_t live_elems = peel_live_elems(nnz);
    SBuf<int32_t> rp, ci;
    CHK(rp.alloc(held, (int64_t)n + 1));
    CHK(ci.alloc(held, nnz));
    hipMemcpyKind kind = ptr_kind == EBBKC_PTR_HOST ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice;
    CHK(hipMemcpyAsync(rp.p, row_ptr, sizeof(int32_t) * ((size_t)n + 1), kind, s));
    if (nnz) CHK(hipMemcpyAsync(ci.p, col_idx, sizeof(int32_t) * (size_t)nnz, kind, s));

    // status words: [0] err, [1] dmax, [2] vertices still uncoloured; read back
    // through the handle's pinned mirror
    if (ebbkc_status st = ensure_counters(g)) return st;
    int* dstat = (int*)g->d_counters;
    int* hstat = (int*)g->h_counters;
    CHK(hipMemsetAsync(dstat, 0, 4 * sizeof(int), s));
    hipLaunchKernelGGL(k_validate_rows, dim3(grid_for((int64_t)n + 1)), dim3(TB), 0, s, rp.p, n, nnz, dstat);
    if (nnz) hipLaunchKernelGGL(k_validate_entries, dim3(grid_for(nnz)), dim3(TB), 0, s, rp.p, ci.p, n, nnz, dstat);
    CHK(hipGetLastError());
    CHK(hipMemcpyAsync(hstat, dstat, sizeof(int), hipMemcpyDeviceToHost, s));
    CHK(hipStreamSynchronize(s));
    if (hstat[0] != 0) return EBBKC_E_BAD_CSR;
    if (nnz % 2 != 0) return EBBKC_E_BAD_CSR;
    const int64_t m = nnz / 2;
    g->m = m;

    // ---- edge ids
    SBuf<int32_t> ustart, ucnt, eid, src, eu, ev;
    SBuf<int64_t> eoff, scan_tmp;
    CHK(ustart.alloc(tmp, n));
    CHK(ucnt.alloc(tmp, n));
    CHK(eoff.alloc(tmp, (int64_t)n + 1));
    CHK(scan_tmp.alloc(tmp, tmp_elems));
    CHK(eid.alloc(tmp, nnz));
    CHK(src.alloc(tmp, nnz));
    CHK(eu.alloc(held, m));
    CHK(ev.alloc(held, m));
    if (n) hipLaunchKernelGGL(k_ustart, dim3(grid_for(n)), dim3(TB), 0, s, rp.p, ci.p, n, ustart.p, ucnt.p, dstat + 1);
    CHK(exclusive_scan_i32(ucnt.p, eoff.p, n, eoff.p + n, scan_tmp.p, s));
    if (nnz)
        hipLaunchKernelGGL(k_edge_ids, dim3(grid_for(nnz)), dim3(TB), 0, s, rp.p, ci.p, n, nnz, ustart.p, eoff.p,
                           eid.p, src.p, eu.p, ev.p);
    CHK(hipGetLastError());

    // ---- degree orientation (id-sorted out rows with edge ids)
    SBuf<int32_t> oflag, orp;
    SBuf<int64_t> opos;
    SBuf<int2> orow_id;
    CHK(oflag.alloc(tmp, nnz));
    CHK(opos.alloc(tmp, nnz));
    CHK(orp.alloc(held, (int64_t)n + 1));
    CHK(orow_id.alloc(tmp, m));
    if (nnz)
        hipLaunchKernelGGL(k_out_flags, dim3(grid_for(nnz)), dim3(TB), 0, s, rp.p, src.p, ci.p, (const int2*)nullptr,
                           nnz, oflag.p);
    CHK(exclusive_scan_i32(oflag.p, opos.p, nnz, nullptr, scan_tmp.p, s));
    hipLaunchKernelGGL(k_out_fill, dim3(grid_for(std::max<int64_t>(nnz, (int64_t)n + 1))), dim3(TB), 0, s, rp.p, ci.p, eid.p,
                       (const int2*)nullptr, n, nnz, oflag.p, opos.p, orow_id.p, orp.p);
    CHK(hipGetLastError());

    // ---- supports and triangle incidence
    SBuf<int32_t> sup, nab, naw, trows;
    SBuf<int64_t> inc_off, cursor;
    CHK(sup.alloc(tmp, m));
    CHK(nab.alloc(tmp, m));
    CHK(naw.alloc(tmp, m));
    CHK(trows.alloc(tmp, 2 + 2 * (int64_t)n));
    CHK(inc_off.alloc(tmp, m + 1));
    CHK(hipMemsetAsync(sup.p, 0, sizeof(int32_t) * (size_t)(m > 0 ? m : 1), s));
    CHK(hipMemsetAsync(trows.p, 0, 2 * sizeof(int32_t), s));
    TriArgs tri{};
    tri.orp = orp.p;
    tri.orow = orow_id.p;
    tri.n = n;
    tri.sup = sup.p;
    tri.nab = nab.p;
    tri.naw = naw.p;
    if (m) {
        hipLaunchKernelGGL(k_tri_rows, dim3(grid_for(n)), dim3(TB), 0, s, orp.p, n, trows.p);
        CHK(launch_tri<0>(tri, trows.p, s));
    }
    CHK(exclusive_scan_i32(sup.p, inc_off.p, m, inc_off.p + m, scan_tmp.p, s));
    int64_t h_ninc = 0;
    CHK(hipMemcpyAsync(g->h_counters + 8, inc_off.p + m, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    CHK(hipMemcpyAsync(hstat + 1, dstat + 1, sizeof(int), hipMemcpyDeviceToHost, s));
    CHK(hipStreamSynchronize(s));
    h_ninc = (int64_t)g->h_counters[8];
    g->max_degree = hstat[1];
    DBuf<int2> inc;
    CHK(inc.alloc(h_ninc));
    CHK(cursor.alloc(tmp, m + 1));
    if (m) {
        hipLaunchKernelGGL(k_tri_cursor, dim3(grid_for(m)), dim3(TB), 0, s, orow_id.p, nab.p, naw.p, inc_off.p, m,
                           (unsigned long long*)cursor.p);
        tri.inc_off = inc_off.p;
        tri.cursor = (unsigned long long*)cursor.p;
        tri.inc = inc.p;
        if (h_ninc) CHK(launch_tri<1>(tri, trows.p, s));
    }
    CHK(hipGetLastError());
    SBuf<int32_t> sup0;
    CHK(sup0.alloc(held, m));
    CHK(hipMemcpyAsync(sup0.p, sup.p, sizeof(int32_t) * (size_t)(m > 0 ? m : 1), hipMemcpyDeviceToDevice, s));

    // ---- level-synchronous peel: rounds, levels and |V(g_i)|, then the ranks
    // by a stable sort of the rounds over the edge ids
    SBuf<int32_t> live, rnd, level, rank, subsize, byrank;
    SBuf<PeelCtl> ctl;
    SBuf<uint32_t> rk1, rk2, rv2;
    SBuf<int64_t> rhist, rtmp;
    const int64_t sorted = nnz;  // the larger of the two sorts that share the buffers
    CHK(level.alloc(held, m));
    CHK(rank.alloc(held, m));
    CHK(subsize.alloc(held, m));
    CHK(byrank.alloc(held, m));
    CHK(rk1.alloc(tmp, sorted));
    CHK(rk2.alloc(tmp, sorted));
    CHK(rv2.alloc(tmp, sorted));
    CHK(rhist.alloc(tmp, radix_hist_elems(sorted)));
    CHK(rtmp.alloc(tmp, rtmp_elems));
    if (m) {
        CHK(rnd.alloc(tmp, m));
        CHK(ctl.alloc(tmp, 1));
        CHK(live.alloc(tmp, live_elems));
        PeelArgs pa{};
        pa.m = (int32_t)m;
        pa.inc_off = inc_off.p;
        pa.inc = inc.p;
        pa.sup = sup.p;
        pa.rnd = rnd.p;
        pa.level = level.p;
        pa.subsize = subsize.p;
        // the triangle pass is through with its places: 8 (m + 1) bytes
        pa.front[0] = (int32_t*)cursor.p;
        pa.front[1] = pa.front[0] + m;
        pa.live = live.p;
        pa.ctl = ctl.p;
        const PeelCtl* hc = (const PeelCtl*)g->h_counters;
        bool fresh = true;  // the supports are those of G
        auto attempt = [&](int64_t grid) -> int {
            const int64_t chunks = (m + PEEL_TB - 1) / PEEL_TB;
            pa.live_chunks = (int32_t)((chunks + grid - 1) / grid);
            if (grid * pa.live_chunks * PEEL_TB > live_elems) return EBBKC_E_HIP;
            if (!fresh) CHK(hipMemcpyAsync(sup.p, sup0.p, sizeof(int32_t) * (size_t)m, hipMemcpyDeviceToDevice, s));
            fresh = false;
            hipLaunchKernelGGL(k_peel_begin, dim3(std::min(grid_for(m), 2048u)), dim3(TB), 0, s, ctl.p, rnd.p,
                               (int32_t)m);
            CHK(hipGetLastError());
            if (grid == 1) {
                hipLaunchKernelGGL(k_peel, dim3(1), dim3(PEEL_TB), 0, s, pa);
                CHK(hipGetLastError());
            } else {
                void* args[] = {&pa};
                if (hipLaunchCooperativeKernel((void*)k_peel, dim3((unsigned)grid), dim3(PEEL_TB), args, 0, s) !=
                    hipSuccess) {
                    (void)hipGetLastError();
                    return PEEL_AGAIN;
                }
            }
            CHK(hipMemcpyAsync(g->h_counters, ctl.p, sizeof(PeelCtl), hipMemcpyDeviceToHost, s));
            CHK(hipStreamSynchronize(s));
            return hc->err ? PEEL_AGAIN : (int)EBBKC_OK;
        };
        const int st = peel_attempts(
            peel_grid(m, peel_resident(g->device, g->cu_count)),
            [](void* f, int64_t grid) { return (*static_cast<decltype(attempt)*>(f))(grid); }, &attempt);
        if (st) return (ebbkc_status)st;
        g->tau = hc->tau;
        g->rounds = hc->rounds;
        // (the sorted ids end in byrank: an odd number of passes starts from the other buffer)
        const int rbits = bits_for((uint64_t)(g->rounds - 1));
        const bool odd = radix_passes(m, rbits) & 1;
        uint32_t* va = odd ? rv2.p : (uint32_t*)byrank.p;
        hipLaunchKernelGGL(k_round_keys, dim3(grid_for(m)), dim3(TB), 0, s, rnd.p, m, rk1.p, va);
        CHK(radix_sort_u32(rk1.p, va, rk2.p, odd ? (uint32_t*)byrank.p : rv2.p, m, rbits, rhist.p, rtmp.p, s, false));
        hipLaunchKernelGGL(k_scatter_pos, dim3(grid_for(m)), dim3(TB), 0, s, (const uint32_t*)byrank.p, m, rank.p);
        CHK(hipGetLastError());
    }

    // ---- root edge order from a vertex order (ablation orderings): edges in the
    // lexicographic order of their endpoints' positions replace pi_tau; levels
    // and tau stay those of the truss peel (tau + 2 still bounds the clique size)
    if ((g->opt.ordering == EBBKC_ORDER_COLOR || g->opt.ordering == EBBKC_ORDER_DEGEN_VERTEX ||
         g->opt.ordering == EBBKC_ORDER_DEGEN_VERTEX_NP) && n > 0) {
        const int64_t big = (int64_t)n > m ? (int64_t)n : m;
        DBuf<int32_t> vpos, vcol;
        DBuf<uint64_t> k1, k2;
        DBuf<uint32_t> v1, v2;
        DBuf<int64_t> rh, rht;
        CHK(vpos.alloc(n));
        CHK(k1.alloc(big));
        CHK(k2.alloc(big));
        CHK(v1.alloc(big));
        CHK(v2.alloc(big));
        const int64_t rhn = radix_hist_elems(big);
        CHK(rh.alloc(rhn));
        CHK(rht.alloc(scan_tmp_elems(rhn) + 16));
        if (g->opt.ordering == EBBKC_ORDER_COLOR) {
            // greedy colouring (Section 4.3), then vertices by colour desc, id asc
            CHK(vcol.alloc(n));
            CHK(hipMemsetAsync(vcol.p, 0, sizeof(int32_t) * (size_t)n, s));
            unsigned gc = grid_for((int64_t)n * EBB_WAVE);
            if (gc > 16384) gc = 16384;
            for (;;) {
                CHK(hipMemsetAsync(dstat + 2, 0, sizeof(int), s));
                hipLaunchKernelGGL(k_colour_round, dim3(gc), dim3(TB), 0, s, rp.p, ci.p, n, vcol.p, dstat + 2);
                CHK(hipGetLastError());
                CHK(hipMemcpyAsync(hstat + 2, dstat + 2, sizeof(int), hipMemcpyDeviceToHost, s));
                CHK(hipStreamSynchronize(s));
                if (hstat[2] == 0) break;
            }
            hipLaunchKernelGGL(k_colour_keys, dim3(grid_for(n)), dim3(TB), 0, s, vcol.p, n, k1.p, v1.p);
            CHK(radix_sort_u64(k1.p, v1.p, k2.p, v2.p, n, 31, rh.p, rht.p, s));
            hipLaunchKernelGGL(k_scatter_pos, dim3(grid_for(n)), dim3(TB), 0, s, v1.p, (int64_t)n, vpos.p);
            CHK(hipGetLastError());
        } else {
            // degeneracy order, level-synchronous: at level s every remaining
            // vertex of degree <= s leaves in one round, placed by (round, id)
            DBuf<int32_t> deg, vlive, vkeep, vfront, vflag, vrnd;
            DBuf<int64_t> vps;
            DBuf<PeelState> st;
            PeelState* hst = (PeelState*)g->h_counters;
            CHK(st.alloc(1));
            CHK(deg.alloc(n));
            CHK(vlive.alloc(n));
            CHK(vkeep.alloc(n));
            CHK(vfront.alloc(n));
            CHK(vflag.alloc(n));
            CHK(vrnd.alloc(n));
            CHK(vps.alloc((int64_t)n + 1));
            hipLaunchKernelGGL(k_degrees, dim3(grid_for(n)), dim3(TB), 0, s, rp.p, n, deg.p);
            hipLaunchKernelGGL(k_iota, dim3(grid_for(n)), dim3(TB), 0, s, vlive.p, (int64_t)n);
            hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n)), dim3(TB), 0, s, vrnd.p, (int64_t)n, -1);
            CHK(hipGetLastError());
            int64_t nl = n, placed = 0;
            int32_t lv = 0, rr = 0;
            while (placed < n) {
                unsigned gl = grid_for(nl, TB * 8);
                if (gl > 2048) gl = 2048;
                hipLaunchKernelGGL(k_peel_reset, dim3(1), dim3(1), 0, s, st.p);
                hipLaunchKernelGGL(k_peel_flag, dim3(gl), dim3(TB), 0, s, vlive.p, nl, deg.p, lv, vflag.p, st.p);
                CHK(exclusive_scan_i32(vflag.p, vps.p, nl, &st.p->nf, scan_tmp.p, s));
                CHK(hipMemcpyAsync(hst, st.p, sizeof(PeelState), hipMemcpyDeviceToHost, s));
                CHK(hipStreamSynchronize(s));
                const int64_t nf = hst->nf;
                if (nf == 0) {
                    lv = hst->minsup;
                    continue;
                }
                hipLaunchKernelGGL(k_peel_compact, dim3(gl), dim3(TB), 0, s, vlive.p, nl, vflag.p, vps.p, vfront.p,
                                   vkeep.p);
                hipLaunchKernelGGL(k_core_assign, dim3(grid_for(nf)), dim3(TB), 0, s, vfront.p, nf, placed, rr,
                                   vpos.p, vrnd.p);
                unsigned gw = grid_for(nf * EBB_WAVE);
                if (gw > 16384) gw = 16384;
                hipLaunchKernelGGL(k_core_remove, dim3(gw), dim3(TB), 0, s, vfront.p, nf, rp.p, ci.p, vrnd.p, deg.p);
                CHK(hipGetLastError());
                placed += nf;
                nl -= nf;
                ++rr;
                int32_t* t = vlive.p; vlive.p = vkeep.p; vkeep.p = t;
            }
        }
        if (m) {
            hipLaunchKernelGGL(k_lex_edge_keys, dim3(grid_for(m)), dim3(TB), 0, s, eu.p, ev.p, vpos.p, m, n, k1.p,
                               v1.p);
            CHK(radix_sort_u64(k1.p, v1.p, k2.p, v2.p, m, bits_for((uint64_t)n * (uint64_t)n), rh.p, rht.p, s));
            hipLaunchKernelGGL(k_scatter_pos, dim3(grid_for(m)), dim3(TB), 0, s, v1.p, m, rank.p);
            CHK(hipMemcpyAsync(byrank.p, v1.p, sizeof(int32_t) * (size_t)m, hipMemcpyDeviceToDevice, s));
            CHK(hipGetLastError());
        }
        g->vpos = vpos.release();
        g->vcol = vcol.release();
    }

    // ---- rank-tagged adjacency
    SBuf<int32_t> erank;
    SBuf<uint32_t> rv1;
    SBuf<int2> rrow, orow;
    CHK(erank.alloc(held, nnz));
    CHK(rv1.alloc(tmp, nnz));
    CHK(rrow.alloc(held, nnz));
    CHK(orow.alloc(held, m));
    if (nnz) {
        hipLaunchKernelGGL(k_erank, dim3(grid_for(nnz)), dim3(TB), 0, s, eid.p, rank.p, nnz, erank.p);
        hipLaunchKernelGGL(k_rrow_keys, dim3(grid_for(m)), dim3(TB), 0, s, byrank.p, eu.p, ev.p, m, rk1.p, rv1.p);
        const int vbits = bits_for((uint64_t)(n - 1));
        CHK(radix_sort_u32(rk1.p, rv1.p, rk2.p, rv2.p, nnz, vbits, rhist.p, rtmp.p, s, false));
        const uint32_t* perm = radix_passes(nnz, vbits) & 1 ? rv2.p : rv1.p;
        hipLaunchKernelGGL(k_gather_rrow, dim3(grid_for(nnz)), dim3(TB), 0, s, perm, byrank.p, eu.p, ev.p, m, rrow.p);
        hipLaunchKernelGGL(k_out_flags, dim3(grid_for(nnz)), dim3(TB), 0, s, rp.p, src.p, ci.p, rrow.p, nnz, oflag.p);
        CHK(exclusive_scan_i32(oflag.p, opos.p, nnz, nullptr, scan_tmp.p, s));
        hipLaunchKernelGGL(k_out_fill, dim3(grid_for(nnz)), dim3(TB), 0, s, rp.p, ci.p, eid.p, rrow.p, n, nnz, oflag.p,
                           opos.p, orow.p, (int32_t*)nullptr);
        CHK(hipGetLastError());
    }
    // ---- adjacency bitmap for sub-branch builds by pair tests (small graphs)
    DBuf<uint64_t> adj;
    DBuf<uint16_t> acum;
    const int32_t amax = g->opt.adj_max_n == 0 ? ADJ_DEFAULT_MAX_N : g->opt.adj_max_n;
    const int32_t aw = (n + 63) / 64;
    const bool with_adj = amax > 0 && n > 0 && n <= amax && m > 0;
    if (with_adj) {
        CHK(adj.alloc((int64_t)n * aw));
        CHK(acum.alloc((int64_t)n * aw));
        CHK(hipMemsetAsync(adj.p, 0, sizeof(uint64_t) * (size_t)n * aw, s));
        hipLaunchKernelGGL(k_adj_fill, dim3(grid_for(nnz)), dim3(TB), 0, s, src.p, ci.p, nnz, aw, adj.p);
        hipLaunchKernelGGL(k_adj_cum, dim3(grid_for((int64_t)n * aw)), dim3(TB), 0, s, rp.p, ci.p, n, aw, acum.p);
    }
    CHK(hipGetLastError());
    CHK(hipEventRecord(ev1, s));
    CHK(hipStreamSynchronize(s));
    float ms = 0.f;
    CHK(hipEventElapsedTime(&ms, ev0, ev1));
    (void)hipEventDestroy(ev0);
    (void)hipEventDestroy(ev1);
    g->prepare_ms = ms;

    g->held = held.release();
    g->rp = rp.p;
    g->ci = ci.p;
    g->erank = erank.p;
    g->eu = eu.p;
    g->ev = ev.p;
    g->sup0 = sup0.p;
    g->rank = rank.p;
    g->level = level.p;
    g->rrow = rrow.p;
    g->orp = orp.p;
    g->orow = orow.p;
    g->byrank = byrank.p;
    g->subsize = subsize.p;  // of pi_tau; another edge order has other sub-branches
    g->subsize_ready = g->opt.ordering == EBBKC_ORDER_HYBRID || g->opt.ordering == EBBKC_ORDER_TRUSS;
    if (with_adj) {
        g->adj = adj.release();
        g->acum = acum.release();
        g->adjw = aw;
    }
    g->device_bytes = (int64_t)sizeof(int32_t) * (((int64_t)n + 1) * 2 + nnz * 2 + m * 7) + (int64_t)sizeof(int2) * (nnz + m) +
                      (int64_t)sizeof(int32_t) * n * ((g->vpos ? 1 : 0) + (g->vcol ? 1 : 0)) +
                      (with_adj ? (int64_t)n * aw * (int64_t)(sizeof(uint64_t) + sizeof(uint16_t)) : 0);
    return EBBKC_OK;
}

}  // namespace ebb
