// build.h -- construction of one sub-branch g_i in LDS by one wavefront,
// shared by the arena builder (which then writes g_i to HBM) and the search
// kernel variant that builds each task's g_i in place (batches too large for
// an arena).
//
// For a seed e_i = (u,v) of rank r (Eq. edge-oriented-branching):
//   1. candidates  V(g_i) = {w : (u,w) and (v,w) both ranked after e_i}.  The
//                  shorter of the two rank-sorted row prefixes (entries ranked
//                  after r) is scanned; each entry is looked up in the other
//                  endpoint's id-sorted row, whose rank must also exceed r.
//   2. sub-graph   E(g_i): pairs of V(g_i) joined by an edge ranked after r.
//                  With an adjacency bitmap of G (small graphs), every pair
//                  of members is tested directly (one bit, and for an edge
//                  its rank found from the bitmap's cumulative counts): about
//                  c^2 / 2 tests, against about c times the out-degree for a
//                  scan.  Otherwise every member's degree-oriented row prefix
//                  ranked after r is streamed, one member at a time over the
//                  wave's lanes, against an LDS hash of V(g_i); each such edge
//                  is met exactly once, and the rows are made symmetric by bit
//                  transposes.  Both give the same rows.
//   3. colouring   greedy colouring (colours 1, 2, ...) visiting vertices by
//                  non-increasing degree in g_i, ties to the smaller vertex
//                  id (Section 4.3; Algorithm EBBkC-H colours each g_i).
//                  Under EBBkC-C the colours of G's own colouring are kept
//                  instead (renumbered 1..D among the colours present).
//   4. order       position of every vertex when sorted by non-increasing
//                  colour, ties to the smaller vertex id (the DAG of
//                  Algorithm EBBkC-H orients edges low -> high in it).
#pragma once
#include "arena.h"
#include "device_util.h"

namespace ebb {

// hash slots: at most a quarter of them taken
template <int W>
constexpr int hash_size() { return W <= 1 ? 256 : (W <= 2 ? 512 : 1024); }
template <int W>
constexpr int hash_bits() { return W <= 1 ? 8 : (W <= 2 ? 9 : 10); }
constexpr uint16_t HASH_FREE = 0xFFFF;

// LDS bytes of the build's work areas (BuildScratch) for width class W
template <int W>
constexpr int build_scratch_bytes() { return 4 * 64 * W + 4 * 64 * W + 2 * hash_size<W>() + 2 * 64 * W; }

template <int W>
__device__ __forceinline__ uint32_t hslot(int32_t key) {
    return ((uint32_t)key * 2654435761u) >> (32 - hash_bits<W>());
}

// The build's LDS work areas: candidate ids, a per-vertex key, the open
// addressing hash (slot -> local index, whose id gid holds) and a visiting
// sequence.
template <int W>
struct BuildScratch {
    int32_t* gid;    // [64 W]
    int32_t* key;    // [64 W]
    uint16_t* hidx;  // [hash_size]
    int16_t* seq;    // [64 W]
    // carve the areas out of `base` (4-byte aligned, build_scratch_bytes<W>() bytes)
    __device__ static BuildScratch carve(void* base) {
        char* p = reinterpret_cast<char*>(base);
        BuildScratch S;
        S.gid = reinterpret_cast<int32_t*>(p);
        p += 4 * 64 * W;
        S.key = reinterpret_cast<int32_t*>(p);
        p += 4 * 64 * W;
        S.hidx = reinterpret_cast<uint16_t*>(p);
        p += 2 * hash_size<W>();
        S.seq = reinterpret_cast<int16_t*>(p);
        return S;
    }
};

// local index of vertex id `key`, or -1
template <int W>
__device__ __forceinline__ int hash_find(const BuildScratch<W>& S, int32_t key) {
    uint32_t h = hslot<W>(key);
    for (;;) {  // some slot is free
        const uint16_t i = S.hidx[h];
        if (i == HASH_FREE) return -1;
        if (S.gid[i] == key) return i;
        h = (h + 1) & (hash_size<W>() - 1);
    }
}

// the c ids of S.gid into the hash: every id tries its slot, the ones that
// find it taken (or lose it to another lane) move on
template <int W>
__device__ __forceinline__ void hash_build(const BuildScratch<W>& S, int c) {
    const int lane = lane_id();
    for (int j = lane; j < hash_size<W>() / 2; j += 64) reinterpret_cast<uint32_t*>(S.hidx)[j] = 0xFFFFFFFFu;
    wave_sync();
    for (int i0 = 0; i0 < c; i0 += 64) {
        const int i = i0 + lane;
        bool wait = i < c;
        uint32_t h = wait ? hslot<W>(S.gid[i]) : 0;
        while (ballot(wait)) {
            const bool try_now = wait && S.hidx[h] == HASH_FREE;
            if (try_now) S.hidx[h] = (uint16_t)i;
            wave_sync();
            if (try_now && S.hidx[h] == (uint16_t)i) wait = false;
            else if (wait) h = (h + 1) & (hash_size<W>() - 1);
            wave_sync();
        }
    }
}

// Whether (x, w) is an edge of G ranked after r: a bit of the adjacency
// bitmap, then the edge's rank at its position in the id-sorted row (the
// entries before its word plus the set bits below it in the word); without
// a bitmap, by binary search of the id-sorted row.
__device__ __forceinline__ bool later_edge(const GraphView& G, int32_t x, int32_t w, int32_t r) {
    if (G.adj) {
        const int64_t o = (int64_t)x * G.adjw + (w >> 6);
        const uint64_t word = G.adj[o];
        if (!((word >> (w & 63)) & 1)) return false;
        return G.erank[G.rp[x] + (int)G.acum[o] + popc64(word & ((1ull << (w & 63)) - 1))] > r;
    }
    const int q = lower_bound_i32(G.ci, G.rp[x], G.rp[x + 1], w);
    return q < G.rp[x + 1] && G.ci[q] == w && G.erank[q] > r;
}

// later_edge for PB pairs (x[t], w[t]) at once: with the bitmap, every load
// of the first step (bitmap word, row start, entries before the word) is
// issued before any is used, then the rank loads of the pairs that are edges,
// so the PB chains of dependent loads overlap instead of following each other.
template <int PB>
__device__ __forceinline__ void later_edges(const GraphView& G, const int32_t (&x)[PB], const int32_t (&w)[PB],
                                            const bool (&valid)[PB], int32_t r, bool (&ok)[PB]) {
    if (G.adj) {
        uint64_t word[PB];
        int32_t row0[PB], below[PB];
#pragma unroll
        for (int t = 0; t < PB; ++t) {
            word[t] = 0;
            row0[t] = 0;
            below[t] = 0;
            if (valid[t]) {
                const int64_t o = (int64_t)x[t] * G.adjw + (w[t] >> 6);
                word[t] = G.adj[o];
                row0[t] = G.rp[x[t]];
                below[t] = (int32_t)G.acum[o];
            }
        }
#pragma unroll
        for (int t = 0; t < PB; ++t) {
            ok[t] = false;
            if (valid[t] && ((word[t] >> (w[t] & 63)) & 1))
                ok[t] = G.erank[row0[t] + below[t] + popc64(word[t] & ((1ull << (w[t] & 63)) - 1))] > r;
        }
    } else {
#pragma unroll
        for (int t = 0; t < PB; ++t) ok[t] = valid[t] && later_edge(G, x[t], w[t], r);
    }
}

// pairs (or row entries) a lane tests per round of the build
constexpr int BUILD_PB = 4;

// Numbers of entries of rows u and v (rank-sorted, descending) ranked after r,
// found by the whole wave: a step loads the last entry of each 64th of what is
// left of either row, so a row of up to 4,096 entries takes two dependent
// loads and the rows are searched side by side (two binary searches one after
// the other, about 18 dependent loads of up to 1 us for rows of 500, were a
// third of a task).
__device__ __forceinline__ void wave_prefixes(const int32_t* __restrict__ rp, const int2* __restrict__ rrow, int32_t u,
                                              int32_t v, int32_t r, int& lu, int& lv) {
    const int lane = lane_id();
    const int bu = uniform_i32(rp[u]), bv = uniform_i32(rp[v]);
    int pu = 0, pv = 0;  // entries known to rank after r; the first n* of the others are undecided
    int nu = uniform_i32(rp[u + 1]) - bu, nv = uniform_i32(rp[v + 1]) - bv;
    while (nu > 0 || nv > 0) {
        const int su = (nu + 63) >> 6, sv = (nv + 63) >> 6;  // entries a lane stands for
        const bool au = lane * su < nu, av = lane * sv < nv;
        int yu = r, yv = r;
        if (au) yu = rrow[bu + pu + min(lane * su + su, nu) - 1].y;
        if (av) yv = rrow[bv + pv + min(lane * sv + sv, nv) - 1].y;
        if (nu > 0) {
            const int full = popc64(ballot(au && yu > r));  // 64ths that are prefix to their last entry
            const int done = min(full * su, nu);
            pu += done;
            nu = min(su, nu - done) - 1;  // the next one's last entry is not
        }
        if (nv > 0) {
            const int full = popc64(ballot(av && yv > r));
            const int done = min(full * sv, nv);
            pv += done;
            nv = min(sv, nv - done) - 1;
        }
    }
    lu = pu;
    lv = pv;
}

// Edges of g_i by streaming the members' degree-oriented rows: rows[j] |= bit
// i for every edge met at member i, one direction only (the lanes of a step
// hold different j, so their LDS updates do not collide), then made symmetric.
// The members are taken one after the other by the whole wave: their offsets
// and prefix lengths are lane values read into scalars, so a step of 64
// entries is a load (issued a step ahead), a hash probe and the update, about
// 30 instructions; VALU-bound.  R-MAT s18 streams 9.1e9 entries for its 3.3 M
// sub-branches: the three classes' builds take 18.0, 11.2 and 6.5 ms (flattening
// all prefixes over the lanes, with a binary search of the member per entry,
// and finding the members again by row searches took 56.6, 57.9 and 33.3 ms).
template <int W>
__device__ __forceinline__ void scan_edges(const GraphView& G, int32_t r, int c, uint64_t (*rows)[W],
                                           const BuildScratch<W>& S) {
    const int lane = lane_id();
    int off[W], len[W];
    {
        // prefixes ranked after r: binary searches of the W members of a lane side by side
        int lo[W], hi[W];
#pragma unroll
        for (int q = 0; q < W; ++q) {
            const int i = lane + 64 * q;
            const int32_t w = i < c ? S.gid[i] : -1;
            off[q] = w >= 0 ? G.orp[w] : 0;
            lo[q] = off[q];
            hi[q] = w >= 0 ? G.orp[w + 1] : 0;
        }
        bool more = true;
        while (more) {
            int y[W];
#pragma unroll
            for (int q = 0; q < W; ++q) y[q] = lo[q] < hi[q] ? G.orow[midpoint(lo[q], hi[q])].y : 0;
            more = false;
#pragma unroll
            for (int q = 0; q < W; ++q) {
                if (lo[q] < hi[q]) {
                    const int mid = midpoint(lo[q], hi[q]);
                    if (y[q] > r) lo[q] = mid + 1; else hi[q] = mid;
                }
                more |= lo[q] < hi[q];
            }
        }
#pragma unroll
        for (int q = 0; q < W; ++q) len[q] = lo[q] - off[q];
    }
#pragma unroll
    for (int q = 0; q < W; ++q) {
        // members with a non-empty prefix
        uint64_t todo = uni64(ballot(len[q] > 0));
        if (!todo) continue;
        int i = __builtin_ctzll(todo);
        todo &= todo - 1;
        int p = __builtin_amdgcn_readlane(off[q], i), e = p + __builtin_amdgcn_readlane(len[q], i);
        int32_t nb = p + lane < e ? G.orow[p + lane].x : -1;
        for (;;) {
            // the step after this one: the member's next 64 entries, or the next member
            const int ci_ = i;
            const int32_t cur = nb;
            bool last = false;
            p += 64;
            if (p >= e) {
                last = todo == 0;
                if (!last) {
                    i = __builtin_ctzll(todo);
                    todo &= todo - 1;
                    p = __builtin_amdgcn_readlane(off[q], i);
                    e = p + __builtin_amdgcn_readlane(len[q], i);
                }
            }
            nb = !last && p + lane < e ? G.orow[p + lane].x : -1;
            if (cur >= 0) {
                const int j = hash_find(S, cur);
                if (j >= 0) atomicOr((unsigned long long*)&rows[j][q], 1ull << ci_);
            }
            if (last) break;
        }
    }
    wave_sync();
    uint64_t T[W][W];
#pragma unroll
    for (int q = 0; q < W; ++q)
#pragma unroll
        for (int w = 0; w < W; ++w) T[q][w] = lane + 64 * q < c ? rows[lane + 64 * q][w] : 0;
    wave_sync();
#pragma unroll
    for (int q = 0; q < W; ++q)
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint64_t t = T[q][w] | transpose64(T[w][q]);
            if (lane + 64 * q < c) rows[lane + 64 * q][w] = t;
        }
}

// Whether a sub-branch of c vertices and twoE / 2 edges goes without colours:
// `plain` says which may.  In a search that does not branch, colours only save
// counting leaves that hold nothing, and they are cheap to count where less
// than half of the pairs are edges; a bipartite sub-branch can reach a half,
// and one of few colours and many edges costs most without them.  32 graphs a
// batch, none / up to a half / all plain, ms: G(200, .4) k = 7 1.13 / 1.03 /
// 1.01, G(150, .5) k = 7 1.30 / 1.27 / 1.25, G(80, .9) k = 6 1.14 / 1.15 / 1.03;
// complete multipartite of 5 x 24 vertices k = 7 1.76 / 1.70 / 4.17, of 6 x 20
// 1.97 / 1.99 / 4.83, of 4 x 30 1.16 / 1.09 / 1.09.
enum : int { PLAIN_NEVER = 0, PLAIN_SPARSE = 1, PLAIN_ALWAYS = 2 };
__device__ __forceinline__ bool plain_build(int plain, int c, uint32_t twoE) {
    return plain == PLAIN_ALWAYS || (plain == PLAIN_SPARSE && 2 * twoE < (uint32_t)c * (uint32_t)c);
}

// Steps 1-3 for the seed (u, v) of rank r (a vertex slot passes u = v and the
// rank threshold of its out-edges): candidates into S.gid -- those given (the
// c = expect members in any order), else found --, their symmetric adjacency
// bitmap into rows (candidate order), colours into col.  Returns c = |V(g_i)|
// (uniform), or -1 when c exceeds 64 W or differs from expect (expect < 0: not
// checked); *twoE = 2 |E(g_i)|.  Without step 3 where plain_build holds.
template <int W>
__device__ int build_subbranch(const GraphView& G, int32_t u, int32_t v, int32_t r, int expect,
                               const int32_t* __restrict__ given, const int32_t* __restrict__ vcol,
                               uint64_t (*rows)[W], int16_t* col, const BuildScratch<W>& S, uint32_t* twoE,
                               int plain = PLAIN_NEVER) {
    const int lane = lane_id();
    constexpr int CAP = 64 * W;

    // ---- 1. candidates
    int c = 0;
    if (given) {
        c = expect;
        if (c > CAP) return -1;
        for (int i = lane; i < c; i += 64) S.gid[i] = given[i];
    } else {
    int lu, lv;
    wave_prefixes(G.rp, G.rrow, u, v, r, lu, lv);
    const int32_t xs = lu <= lv ? u : v, ys = lu <= lv ? v : u;
    const int lx = lu <= lv ? lu : lv;
    const int32_t xrow = G.rp[xs];
    for (int base = 0; base < lx; base += 64 * BUILD_PB) {
        int32_t wv[BUILD_PB], yv[BUILD_PB];
        bool val[BUILD_PB], okv[BUILD_PB];
#pragma unroll
        for (int t = 0; t < BUILD_PB; ++t) {
            const int idx = base + 64 * t + lane;
            val[t] = idx < lx;
            wv[t] = val[t] ? G.rrow[xrow + idx].x : -1;
            yv[t] = ys;
        }
        later_edges<BUILD_PB>(G, yv, wv, val, r, okv);
#pragma unroll
        for (int t = 0; t < BUILD_PB; ++t) {  // in row order, as one entry per lane per round
            const uint64_t mk = ballot(okv[t]);
            if (okv[t]) {
                const int p = c + popc64(mk & lanemask_lt());
                if (p < CAP) S.gid[p] = wv[t];
            }
            c += popc64(mk);
        }
    }
    }
    c = uniform_i32(c);
    if (c > CAP || (expect >= 0 && c != expect)) return -1;

    // ---- 2. sub-graph bitmap
    for (int i = lane; i < c; i += 64)
#pragma unroll
        for (int w = 0; w < W; ++w) rows[i][w] = 0;
    if (G.adj) {
        for (int i = lane; i < c; i += 64) S.key[i] = G.rp[S.gid[i]];
        wave_sync();
        // the pairs (i, j), i < j, two rows folded to c pairs: fold a holds row a
        // (c - 1 - a pairs), then row c - 2 - a (a + 1 pairs), so an index needs
        // no root and the lanes of a step read few rows of the bitmap (ten
        // graphs of up to 5,000 vertices, every task building: 43 ms; 49 with the
        // row found from a square root, 56 with 64 different rows a step)
        const int U = c * (c - 1) / 2;
        const float inv = 1.0f / (float)c;
        for (int u0 = 0; u0 < U; u0 += 64 * BUILD_PB) {
            int pi[BUILD_PB], pj[BUILD_PB];
            uint64_t word[BUILD_PB], bit[BUILD_PB];
            int32_t pos[BUILD_PB];
#pragma unroll
            for (int t = 0; t < BUILD_PB; ++t) {
                const int u = u0 + 64 * t + lane;
                const int fold = (int)(((float)u + 0.5f) * inv);  // u / c: exact below 2^16
                const int b = u - fold * c;
                const bool first = b < c - 1 - fold;
                pi[t] = first ? fold : c - 2 - fold;
                pj[t] = first ? fold + 1 + b : b;
                word[t] = 0;
                bit[t] = 0;
                pos[t] = 0;
                if (u < U) {
                    const int32_t w = S.gid[pj[t]];
                    const int64_t o = (int64_t)S.gid[pi[t]] * G.adjw + (w >> 6);
                    word[t] = G.adj[o];
                    pos[t] = S.key[pi[t]] + (int32_t)G.acum[o];
                    bit[t] = 1ull << (w & 63);
                }
            }
#pragma unroll
            for (int t = 0; t < BUILD_PB; ++t) {
                int32_t rk = -1;
                if (word[t] & bit[t]) rk = G.erank[pos[t] + popc64(word[t] & (bit[t] - 1))];
                pos[t] = rk;
            }
#pragma unroll
            for (int t = 0; t < BUILD_PB; ++t) {
                if (pos[t] > r) {
                    atomicOr((unsigned long long*)&rows[pi[t]][pj[t] >> 6], 1ull << (pj[t] & 63));
                    atomicOr((unsigned long long*)&rows[pj[t]][pi[t] >> 6], 1ull << (pi[t] & 63));
                }
            }
        }
    } else {
        wave_sync();
        hash_build(S, c);
        scan_edges(G, r, c, rows, S);
    }
    wave_sync();

    // ---- 3a. colouring order: degree desc, id asc
    uint32_t dsum = 0;
#pragma unroll
    for (int q = 0; q < W; ++q) {
        const int i = lane + 64 * q;
        if (i < c) {
            int d = 0;
#pragma unroll
            for (int w = 0; w < W; ++w) d += popc64(rows[i][w]);
            S.key[i] = d;
            dsum += d;
        }
    }
    *twoE = wave_sum(dsum);
    wave_sync();
    if (plain_build(plain, c, *twoE)) return c;
    if (vcol) {
        // ---- 3'. G's colouring kept (EBBkC-C): the colours present are
        // renumbered 1..D in their order, which changes neither the order
        // below nor the number of colours in any vertex set
        for (int i = lane; i < c; i += 64) S.key[i] = vcol[S.gid[i]];
        wave_sync();
#pragma unroll
        for (int q = 0; q < W; ++q) {
            const int i = lane + 64 * q;
            const int ki = i < c ? S.key[i] : 0, gi = i < c ? S.gid[i] : 0;
            int ord = 0;
            for (int j = 0; j < c; ++j) {
                const int kj = S.key[j], gj = S.gid[j];
                ord += (kj > ki) || (kj == ki && gj < gi);
            }
            if (i < c) S.seq[ord] = (int16_t)i;
        }
        wave_sync();
        int cum[W];
        int starts = 0;
#pragma unroll
        for (int q = 0; q < W; ++q) {
            const int p = lane + 64 * q;
            const bool st = p < c && (p == 0 || S.key[S.seq[p]] != S.key[S.seq[p - 1]]);
            const uint64_t mk = ballot(st);
            cum[q] = starts + popc64(mk & (lanemask_lt() | (1ull << lane)));
            starts += popc64(mk);
        }
#pragma unroll
        for (int q = 0; q < W; ++q) {
            const int p = lane + 64 * q;
            if (p < c) col[S.seq[p]] = (int16_t)(starts - cum[q] + 1);
        }
        wave_sync();
    } else {
#pragma unroll
        for (int q = 0; q < W; ++q) {
            const int i = lane + 64 * q;
            const int di = i < c ? S.key[i] : 0, gi = i < c ? S.gid[i] : 0;
            int ord = 0;
            for (int j = 0; j < c; ++j) {
                const int dj = S.key[j], gj = S.gid[j];
                ord += (dj > di) || (dj == di && gj < gi);
            }
            if (i < c) S.seq[ord] = (int16_t)i;
        }
        wave_sync();
        // ---- 3b. greedy colouring; colour-class masks live in lanes
        uint64_t cls[W][W];
#pragma unroll
        for (int q = 0; q < W; ++q)
#pragma unroll
            for (int w = 0; w < W; ++w) cls[q][w] = 0;
        int ncol = 0;
        for (int t = 0; t < c; ++t) {
            const int i = S.seq[t];
            uint64_t A[W];
#pragma unroll
            for (int w = 0; w < W; ++w) A[w] = rows[i][w];
            int found = -1;
#pragma unroll
            for (int q = 0; q < W; ++q) {
                bool ok = lane + 64 * q < ncol;
#pragma unroll
                for (int w = 0; w < W; ++w) ok = ok && ((cls[q][w] & A[w]) == 0);
                const uint64_t mk = ballot(ok);
                if (found < 0 && mk) found = 64 * q + __builtin_ctzll(mk);
            }
            if (found < 0) found = ncol++;
            found = uniform_i32(found);
            if (lane == (found & 63)) {
#pragma unroll
                for (int q = 0; q < W; ++q)
                    if (q == (found >> 6)) {
#pragma unroll
                        for (int w = 0; w < W; ++w)
                            if (w == (i >> 6)) cls[q][w] |= 1ull << (i & 63);
                    }
            }
            if (lane == 0) col[i] = (int16_t)(found + 1);
        }
        wave_sync();
    }
    return c;
}

// Step 4: npos[q] = position of local vertex lane + 64 q in the order by
// non-increasing colour, ties to the smaller global id (also stored in S.key).
template <int W>
__device__ __forceinline__ void order_positions(int c, const int16_t* col, const BuildScratch<W>& S, int (&npos)[W]) {
    const int lane = lane_id();
#pragma unroll
    for (int q = 0; q < W; ++q) {
        const int i = lane + 64 * q;
        const int ci_ = i < c ? col[i] : 0, gi = i < c ? S.gid[i] : 0;
        int ord = 0;
        for (int j = 0; j < c; ++j) {
            const int cj = col[j], gj = S.gid[j];
            ord += (cj > ci_) || (cj == ci_ && gj < gi);
        }
        npos[q] = ord;
        if (i < c) S.key[i] = ord;
    }
    wave_sync();
}

// Row of local vertex i with its bits moved to the vertices' positions
template <int W>
__device__ __forceinline__ void relabelled_row(const uint64_t (*rows)[W], int i, const BuildScratch<W>& S,
                                               uint64_t (&nr)[W]) {
#pragma unroll
    for (int w = 0; w < W; ++w) nr[w] = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        uint64_t b = rows[i][w];
        while (b) {
            const int j = w * 64 + __builtin_ctzll(b);
            b &= b - 1;
            const int pj = S.key[j];
#pragma unroll
            for (int ww = 0; ww < W; ++ww)
                if (ww == (pj >> 6)) nr[ww] |= 1ull << (pj & 63);
        }
    }
}

}  // namespace ebb
