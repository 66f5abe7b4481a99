// search_kernel.h -- the EBBkC-C_Rec search over arena sub-branches (one
// wavefront per task).
//
// A task is a seed's g_i (from the arena, or built in LDS by the task) and a
// range of first vertices of the root's children; light seeds are
// one task, heavy seeds one task per range of root vertices.  While some
// waves wait for work, a node can also be handed to one of them through a
// device queue.  On the DAG of g_i (vertices in colour order, edges
// low -> high) a node (P, l):
//   * is pruned when |P| < l (Algorithm EBBkC);
//   * at l = 1 counts |P|, at l = 2 the edges inside P;
//   * at l >= 3 is finished in closed form when P is a clique, C(|P|, l), or
//     a 2-plex, sum_j C(p, j) 2^j C(f, l-j) with f full vertices and p
//     non-adjacent pairs (Section 5, Algorithm kC2Plex);
//   * at l = 3 counts the triangles inside P;
//   * otherwise branches on every DAG edge x->y inside P into
//     P' = P & N+(x) & N+(y), l-2, skipping children by Rule (1)
//     (col x < l or col y < l-1) and Rule (2) (fewer than l-2 colours in P')
//     (Section 4.3, Algorithm EBBkC-C).
// Nodes with l = 4 or 5 hand their children (l = 2 or 3) to lanes, one child
// per lane, after renumbering onto one word fewer when the node's candidate
// set fits; everything above is wave-uniform with the lanes owning rows.
//
// Included by one source per width class (search_w1.hip .. search_w4.hip), so
// that the classes compile side by side, and by search.hip, which instantiates
// none of it.
#pragma once
#include <atomic>
#include <type_traits>

#include "arena.h"
#include "binom.h"
#include "build.h"
#include "device_util.h"

namespace ebb {

namespace {

// l-cliques of a 2-plex with f vertices adjacent to all others and p
// non-adjacent pairs: sum_j C(p,j) 2^j C(f, l-j), exactly in 128 bits
__device__ u128 twoplex_count(int f, int p, int l, bool& ovf) {
    u128 s = 0;
    const int jmax = p < l ? p : l;
    for (int j = 0; j <= jmax; ++j) {
        if (l - j > f) continue;
        u128 t = mul128(binom128(p, j, ovf), binom128(f, l - j, ovf), ovf);
        if (t == 0) continue;
        if (j >= 128 || (t >> (127 - j)) != 0) { ovf = true; return 0; }
        t <<= j;
        s += t;
        if (s < t) { ovf = true; return 0; }
    }
    return s;
}

// exact 128-bit accumulator with an overflow flag, of wave-uniform values:
// they come from table loads and lane sums, which the compiler would keep, and
// the accumulators with them, in vector registers
struct Acc {
    u128 v;
    bool ovf;
    __device__ void add(u128 x) {
        x = ((u128)uni64((uint64_t)(x >> 64)) << 64) | uni64((uint64_t)x);
        v += x;
        ovf |= v < x;
    }
    __device__ uint64_t lo() const { return (uint64_t)v; }
    __device__ uint64_t hi() const { return (uint64_t)(v >> 64); }
};

// the same in 64 bits, for tasks that cannot pass them
struct Acc64 {
    uint64_t v;
    bool ovf;
    __device__ void add(uint64_t x) { v += uni64(x); }
    __device__ uint64_t lo() const { return v; }
    __device__ uint64_t hi() const { return 0; }
};

// twoplex_count for l <= 5 and at most 256 vertices, in 64 bits
__device__ __forceinline__ uint64_t twoplex_small(int f, int p, int l) {
    uint64_t s = 0;
    for (int j = 0; j <= l; ++j) s += binom(p, j) * binom(f, l - j) << j;
    return s;
}

template <int W>
struct Frame {
    uint64_t P[W];
    uint64_t R[W];
    int32_t x, l, y, pad;
};

// children queued per node before the lanes count them (room for one more x)
constexpr int QRUN = 256, QCAP = QRUN + 256;
// W = 1: candidate sets queued per task (room for 64 more), and the least
// |P & N+(x)| of an l = 5 node whose 4-cliques may be taken by the wave: the
// matrix cores take a set in much the same time whatever its size, the queue's
// lanes in time that grows with its pairs.  With 8 / 12 / 16 / 24 / 65 (never),
// ms: R-MAT s16 k = 7 13.4 / 13.3 / 13.2 / 13.1 / 15.6, s13 k = 9 12.3 / 11.8 /
// 11.2 / 10.4 / 10.8; planted cliques on 300,000 vertices k = 7 1.71 / 1.64 /
// 1.63 / 1.60 / 1.52, k = 9 17.8 / 16.1 / 15.0 / 14.2 / 13.7.
constexpr int Q1_CAP = 256, Q1_RUN = Q1_CAP - 64, L5_WAVE_MIN = 24;

template <int W>
struct SearchMem {
    uint64_t rows[64 * W][W];
    uint64_t dag[W == 1 ? 64 : 1];  // W = 1: the later neighbours of each vertex
    int32_t pushed;                 // this wave handed a node over in this launch
    int16_t col[64 * W];
    int16_t md[64 * W];      // missing pairs per vertex inside the set being counted
    int16_t vl[64 * W];      // that set's vertices in order, one per lane
    // queued children |Q| << 16 | x << 8 | y (and a sort buffer), also the closed
    // forms' work area (all that W = 1 needs it for)
    alignas(16) int32_t pq[2][W == 1 ? 260 : QCAP];
    uint64_t q1[W == 1 ? 2 : 1][W == 1 ? Q1_CAP : 1];  // W = 1: queued candidate sets, and a sort buffer
    Frame<W> fr[LDS_FRAMES];
    // a node's candidate set renumbered onto W - 1 words (compact_set, W = 2
    // and 3): rows of up to 64 (W - 1) vertices, and their colours
    uint64_t crow[W == 2 || W == 3 ? 64 * (W - 1) * (W - 1) : 1];
    int16_t ccol[W == 2 || W == 3 ? 64 * (W - 1) : 1];
};

// nodes with fewer candidates are not renumbered onto narrower rows
constexpr int COMPACT_MIN = 16;

// The p vertices of P (p <= 64 WV, WV < W) renumbered 0 .. p-1 in ascending
// order, with their rows restricted to P and renumbered likewise (WV words)
// and their colours.  The order is kept, so the DAG (lower index first), the
// colour order and every clique inside P are the same; the node's leaves
// then run on WV-word rows.
template <int W, int WV>
__device__ void compact_set(const SearchMem<W>& M, const uint64_t (&P)[W], uint64_t (*rows_out)[WV],
                            int16_t* col_out) {
    const int lane = lane_id();
    int base = 0;
#pragma unroll
    for (int q = 0; q < W; ++q) {
        if (!P[q]) continue;
        if ((P[q] >> lane) & 1) {
            const int v = 64 * q + lane;
            const int idx = base + popc64(P[q] & lanemask_lt());
            uint64_t nr[WV];
#pragma unroll
            for (int z = 0; z < WV; ++z) nr[z] = 0;
            uint64_t cur = 0;
            int t = 0;
#pragma unroll
            for (int qq = 0; qq < W; ++qq) {
                const uint64_t rw = M.rows[v][qq];
                uint64_t bq = P[qq];
                while (bq) {
                    const int b = __builtin_ctzll(bq);
                    bq &= bq - 1;
                    cur |= ((rw >> b) & 1ull) << (t & 63);
                    if ((t & 63) == 63) {
#pragma unroll
                        for (int z = 0; z < WV; ++z)
                            if (z == (t >> 6)) nr[z] = cur;
                        cur = 0;
                    }
                    ++t;
                }
            }
            if (t & 63) {
#pragma unroll
                for (int z = 0; z < WV; ++z)
                    if (z == (t >> 6)) nr[z] = cur;
            }
#pragma unroll
            for (int z = 0; z < WV; ++z) rows_out[idx][z] = nr[z];
            col_out[idx] = M.col[v];
        }
        base += popc64(P[q]);
    }
    wave_sync();
}

// ---------------------------------------------------------------- per-lane leaves
// One lane counts the cliques of one child candidate set Q from LDS rows.

template <int W>
__device__ __forceinline__ uint64_t lane_edges(const uint64_t (*rows)[W], const uint64_t (&Q)[W]) {
    uint32_t e2 = 0;
#pragma unroll
    for (int wz = 0; wz < W; ++wz) {
        uint64_t bits = Q[wz];
        while (bits) {
            const int z = wz * 64 + __builtin_ctzll(bits);
            bits &= bits - 1;
#pragma unroll
            for (int w = 0; w < W; ++w) e2 += popc64(Q[w] & rows[z][w]);
        }
    }
    return e2 / 2;
}

// W = 1: edges and triangles inside Q along the DAG rows
__device__ __forceinline__ uint32_t lane_edges1(const uint64_t* dag, uint64_t Q) {
    uint32_t e = 0;
    while (Q) {
        const int z = __builtin_ctzll(Q);
        Q &= Q - 1;
        e += popc64(Q & dag[z]);
    }
    return e;
}

// Triangles inside Q.  Dense Q (missing pairs M <= edges E): T = C(q,3) -
// M(q-2) + sum_v C(m_v,2) - T_c with m_v the missing pairs at v and T_c the
// triangles of missing pairs; sparse Q: common out-neighbours along the DAG
// edges.  dense_hint (the parent set is dense, so Q almost surely is) takes
// the degrees and T_c in one pass over Q with 32-bit bit iteration, and falls
// back to the sparse pass if Q turns out sparse after all; otherwise the
// degrees come first and only the needed pass follows.
template <int W>
__device__ __forceinline__ uint64_t lane_triangles(const uint64_t (*rows)[W], const uint64_t (&Q)[W], bool dense_hint,
                                                   uint64_t& ops) {
    constexpr int H = 2 * W;  // 32-bit halves of a row
    const int q = popcW(Q);
    if (q < 3) return 0;
    const uint64_t q64 = (uint64_t)q;
    const uint64_t C3 = q64 * (q64 - 1) * (q64 - 2) / 6;
    uint32_t e2 = 0, s2 = 0, t = 0;
    if (dense_hint) {
        uint32_t Qh[H];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            Qh[2 * w] = (uint32_t)Q[w];
            Qh[2 * w + 1] = (uint32_t)(Q[w] >> 32);
        }
#pragma unroll
        for (int hz = 0; hz < H; ++hz) {
            uint32_t bits = Qh[hz];
            while (bits) {
                const int b = __builtin_ctz(bits);
                bits &= bits - 1;
                const uint32_t* rz = reinterpret_cast<const uint32_t*>(rows[32 * hz + b]);
                uint32_t Cz[H];  // missing pairs z-y inside Q with y > z
                int d = 0;
#pragma unroll
                for (int g = 0; g < H; ++g) {
                    const uint32_t row = rz[g];
                    d += __builtin_popcount(Qh[g] & row);
                    if (g > hz) Cz[g] = Qh[g] & ~row;
                    else if (g == hz) Cz[g] = Qh[g] & ~row & (b == 31 ? 0u : (~0u << (b + 1)));
                    else Cz[g] = 0;
                }
                e2 += d;
                const int cm = q - 1 - d;
                s2 += (uint32_t)(cm * (cm - 1) / 2);
#pragma unroll
                for (int gy = hz; gy < H; ++gy) {
                    while (Cz[gy]) {
                        const uint32_t* ry = reinterpret_cast<const uint32_t*>(rows[32 * gy + __builtin_ctz(Cz[gy])]);
                        Cz[gy] &= Cz[gy] - 1;
#pragma unroll
                        for (int g = gy; g < H; ++g) t += __builtin_popcount(Cz[g] & ~ry[g]);
                    }
                }
            }
        }
        const uint64_t Mp = (q64 * (q64 - 1) - e2) / 2, E = e2 / 2;
        ops += (uint64_t)q * W;
        if (Mp == 0) return C3;
        if (Mp <= E) {
            ops += Mp * W;
            return C3 - Mp * (q64 - 2) + s2 - t;
        }
        t = 0;  // sparse after all: the pass along edges below
    } else {
#pragma unroll
        for (int wz = 0; wz < W; ++wz) {
            uint64_t bits = Q[wz];
            while (bits) {
                const int z = wz * 64 + __builtin_ctzll(bits);
                bits &= bits - 1;
                int d = 0;
#pragma unroll
                for (int w = 0; w < W; ++w) d += popc64(Q[w] & rows[z][w]);
                e2 += d;
                const int cm = q - 1 - d;
                s2 += (uint32_t)(cm * (cm - 1) / 2);
            }
        }
        ops += (uint64_t)q * W;
    }
    const uint64_t Mp = (q64 * (q64 - 1) - e2) / 2, E = e2 / 2;
    if (Mp == 0) return C3;
    const bool dense = Mp <= E;
    ops += (dense ? Mp : E) * W;
#pragma unroll
    for (int wz = 0; wz < W; ++wz) {
        uint64_t bits = Q[wz];
        while (bits) {
            const int z = wz * 64 + __builtin_ctzll(bits);
            bits &= bits - 1;
            uint64_t Cz[W];  // missing (dense) or present (sparse) pairs z-y, y > z, inside Q
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const uint64_t row = dense ? ~rows[z][w] : rows[z][w];
                Cz[w] = Q[w] & row & upper_mask(z, w);
            }
#pragma unroll
            for (int wy = 0; wy < W; ++wy) {
                while (Cz[wy]) {
                    const int y = wy * 64 + __builtin_ctzll(Cz[wy]);
                    Cz[wy] &= Cz[wy] - 1;
#pragma unroll
                    for (int w = 0; w < W; ++w) {
                        const uint64_t row = dense ? ~rows[y][w] : rows[y][w];
                        if (w >= wy) t += popc64(Cz[w] & row);
                    }
                }
            }
        }
    }
    return dense ? C3 - Mp * (q64 - 2) + s2 - t : (uint64_t)t;
}

// H = the missing pairs of R, self pairs included.  The sum of the squares of
// all entries of the matrix product H H (codegrees; self pairs add 2 to a
// missing pair's, 1 to a diagonal entry): each lane returns its part.  The
// product is formed by the matrix cores in 16 x 16 tiles: a lane holds 16 bits
// of a row of H as bytes (row lane mod 16 of a block of 16 of R's vertices,
// columns 16 (lane / 16) .. + 15 of a 64-column word of the sub-branch), the
// same fragment serves as either operand, and only the sum of the squares of
// the tile's entries is needed, so no lane needs to know which entry it holds.
// Tiles above the diagonal count twice.  vl: R's r vertices in order.  (A lane
// walking the 2-paths of its vertices took a word operation for each: R-MAT
// s18 at k = 7 306 ms and k = 8 8.52 s, against 180 ms and 4.78 s with the
// matrix cores and each missing pair taken at one end only.)
typedef int v4i __attribute__((ext_vector_type(4)));

template <int WV>
__device__ __forceinline__ v4i missing_fragment(const uint64_t (&R)[WV], const uint64_t (*rows)[WV], int v, int kb) {
    const int g = lane_id() >> 4;
    uint32_t h = 0;
    if (v >= 0) h = (uint32_t)(R[kb] >> (16 * g)) & ~(uint32_t)reinterpret_cast<const uint16_t*>(rows[v])[4 * kb + g];
    v4i f;  // bit k of h to byte k: a nibble times 1 + 2^7 + 2^14 + 2^21
#pragma unroll
    for (int n = 0; n < 4; ++n) f[n] = (int)(__umul24((h >> (4 * n)) & 15u, 0x204081u) & 0x01010101u);
    return f;
}

// GI row blocks are held at a time: four in the shallow kernels of up to two
// words (R-MAT s18 at k = 7, two words 71.4 ms, with two 73.7), two in the deep
// ones, which have fewer registers left (with four they kept 344 bytes a lane in
// scratch at two words, now 220).
template <int WV, int GI>
__device__ __forceinline__ uint32_t codegree_squares(const uint64_t (&R)[WV], const uint64_t (*rows)[WV],
                                                     const int16_t* vl, int r) {
    const int row = lane_id() & 15;
    const int nb = (r + 15) >> 4;
    uint32_t sum = 0;
    auto load = [&](int blk, v4i (&f)[WV]) {
        const int a = 16 * blk + row;
        const int v = a < r ? vl[a] : -1;
#pragma unroll
        for (int kb = 0; kb < WV; ++kb)
            if (R[kb]) f[kb] = missing_fragment<WV>(R, rows, v, kb);
    };
    auto tile = [&](const v4i (&x)[WV], const v4i (&y)[WV]) -> uint32_t {
        v4i c = {0, 0, 0, 0};
#pragma unroll
        for (int kb = 0; kb < WV; ++kb)
            if (R[kb]) c = __builtin_amdgcn_mfma_i32_16x16x64_i8(x[kb], y[kb], c, 0, 0, 0);
        uint32_t q = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) q += __umul24((uint32_t)c[e], (uint32_t)c[e]);
        return q;
    };
    for (int i0 = 0; i0 < nb; i0 += GI) {
        v4i fi[GI][WV];
#pragma unroll
        for (int g = 0; g < GI; ++g) {
            if (i0 + g >= nb) break;
            load(i0 + g, fi[g]);
#pragma unroll
            for (int h = 0; h < GI; ++h)
                if (h <= g) sum += (h < g ? 2 : 1) * tile(fi[h], fi[g]);
        }
        for (int j = i0 + GI; j < nb; ++j) {
            v4i fj[WV];
            load(j, fj);
#pragma unroll
            for (int g = 0; g < GI; ++g) sum += 2 * tile(fi[g], fj);
        }
    }
    return sum;
}

// l-cliques of a 3-plex P (every vertex misses at most two others of P):
// the coefficient of x^l in the independence polynomial of the missing
// pairs H[P], a disjoint union of paths and cycles; Algorithm kCtPlex
// reaches the same sets by branching on H.  Lanes walk the components from
// their vertices into length histograms; the product of path polynomials
// (sum_i C(L-i+1, i) x^i) and cycle polynomials (sum_i [C(L-i, i) +
// C(L-i-1, i-1)] x^i) is formed in LDS, lane j mod 64 owning coefficient j.
// Needs l < pc (so l < 256); sets ovf when the coefficient reaches 2^128.
template <int W>
__device__ __forceinline__ u128 threeplex_count(SearchMem<W>& M, const uint64_t (&P)[W], int pc, int l, bool& ovf) {
const int lane = lane_id();
        int32_t* hp = M.pq[0];   // paths by length
        int32_t* hcy = M.pq[1];  // cycles by length
        for (int i = lane; i < 257; i += 64) { hp[i] = 0; hcy[i] = 0; }
        {
            int base = 0;
#pragma unroll
            for (int q = 0; q < W; ++q) {
                if ((P[q] >> lane) & 1) M.vl[base + popc64(P[q] & lanemask_lt())] = (int16_t)(lane + 64 * q);
                base += popc64(P[q]);
            }
        }
        wave_sync();
        const int rounds = (pc + 63) >> 6;
        for (int t = 0; t < rounds; ++t) {
            const int j = 64 * t + lane;
            if (j < pc) {
                const int v = M.vl[j];
                int mv = -1;  // P & ~row(v) holds v itself
#pragma unroll
                for (int w = 0; w < W; ++w) mv += popc64(P[w] & ~M.rows[v][w]);
                M.md[v] = (int16_t)mv;
            }
        }
        wave_sync();
        // an H-neighbour of cur other than avoid (-1: none)
        auto hnext = [&](int cur, int avoid) -> int {
            int r = -1;
#pragma unroll
            for (int w = W - 1; w >= 0; --w) {
                uint64_t h = P[w] & ~M.rows[cur][w];
                if (w == (cur >> 6)) h &= ~(1ull << (cur & 63));
                if (avoid >= 0 && w == (avoid >> 6)) h &= ~(1ull << (avoid & 63));
                if (h) r = w * 64 + __builtin_ctzll(h);
            }
            return r;
        };
        for (int t = 0; t < rounds; ++t) {
            const int j = 64 * t + lane;
            if (j >= pc) continue;
            const int v = M.vl[j];
            const int mv = M.md[v];
            if (mv <= 1) {  // end of a path (or a lone vertex): walk to the other end
                int prev = -1, cur = v, L = 1;
                if (mv == 1) {
                    for (;;) {
                        const int nx = hnext(cur, prev);
                        prev = cur;
                        cur = nx;
                        ++L;
                        if (M.md[cur] <= 1) break;
                    }
                }
                if (mv == 0 || v < cur) atomicAdd(&hp[L], 1);
            } else {  // on a cycle if the walk comes back to v without meeting an end
                int prev = v, cur = hnext(v, -1), L = 1, mn = v;
                bool cyc = true;
                while (cur != v) {
                    if (M.md[cur] <= 1) { cyc = false; break; }
                    mn = cur < mn ? cur : mn;
                    const int nx = hnext(cur, prev);
                    prev = cur;
                    cur = nx;
                    ++L;
                }
                if (cyc && mn == v) atomicAdd(&hcy[L], 1);
            }
        }
        wave_sync();
        // the histograms move to md / vl (component length L at index L - 1,
        // L <= pc <= 64 W) so that pq can hold the product's coefficients
        for (int L = 1 + lane; L <= pc; L += 64) {
            M.md[L - 1] = (int16_t)hp[L];
            M.vl[L - 1] = (int16_t)hcy[L];
        }
        wave_sync();
        // coefficient j = lane + 64 q of the running product lives at poly[j]
        // (degrees 0..l, l <= 255); a coefficient that reached 2^128 is
        // flagged in the wave-uniform bit set fl and stays flagged, since
        // every factor has positive coefficients up to its degree
        u128* poly = reinterpret_cast<u128*>(&M.pq[0][0]);
        const int Q = (l >> 6) + 1;
#pragma unroll
        for (int q = 0; q < W; ++q)
            if (q < Q) poly[lane + 64 * q] = (lane + 64 * q == 0) ? (u128)1 : (u128)0;
        uint64_t fl[W];
#pragma unroll
        for (int q = 0; q < W; ++q) fl[q] = 0;
        wave_sync();
        auto flagged = [&](int j) -> bool {
            bool f = false;
#pragma unroll
            for (int q = 0; q < W; ++q)
                if ((j >> 6) == q) f = (fl[q] >> (j & 63)) & 1;
            return f;
        };
        // poly <- poly * sum_{i <= deg} coef(i) x^i, truncated at degree l
        auto mulpoly = [&](int deg, auto coef) {
            u128 nr[W];
            bool no[W];
#pragma unroll
            for (int q = 0; q < W; ++q) { nr[q] = 0; no[q] = false; }
            const int imax = deg < l ? deg : l;
            for (int i = 0; i <= imax; ++i) {
                bool co = false;
                const u128 c = coef(i, co);
#pragma unroll
                for (int q = 0; q < W; ++q) {
                    const int j = lane + 64 * q;
                    if (q >= Q || j > l || j < i || no[q]) continue;
                    if (flagged(j - i)) { no[q] = true; continue; }
                    const u128 o = poly[j - i];
                    if (!o) continue;
                    if (co) { no[q] = true; continue; }
                    bool mo = false;
                    const u128 t = mul128(c, o, mo);
                    nr[q] += t;
                    no[q] = mo || nr[q] < t;
                }
            }
            wave_sync();
#pragma unroll
            for (int q = 0; q < W; ++q) {
                if (q < Q) poly[lane + 64 * q] = nr[q];
                fl[q] |= uni64(__ballot(no[q]));
            }
            wave_sync();
        };
        for (int L = 1; L <= pc; ++L) {
            const int np = M.md[L - 1], nc = M.vl[L - 1];
            if (np && L == 1) {
                mulpoly(np, [&](int i, bool& o) { return binom128(np, i, o); });
            } else if (np && L == 2) {
                mulpoly(np, [&](int i, bool& o) {
                    if (i >= 128) { o = true; return (u128)0; }
                    return mul128(binom128(np, i, o), (u128)1 << i, o);
                });
            } else {
                for (int rep = 0; rep < np; ++rep)
                    mulpoly((L + 1) / 2, [&](int i, bool& o) { return binom128(L - i + 1, i, o); });
            }
            for (int rep = 0; rep < nc; ++rep)
                mulpoly(L / 2, [&](int i, bool& o) {
                    if (i == 0) return (u128)1;
                    const u128 x = binom128(L - i, i, o), y = binom128(L - i - 1, i - 1, o);
                    if (x + y < x) o = true;
                    return x + y;
                });
        }
        ovf |= flagged(l);
        const u128 res = poly[l];
        wave_sync();
        return res;
}

// l-cliques of a t-plex P (every vertex misses at most t-1 others of P),
// any t, by Algorithm kCtPlex: the vertices adjacent to all others (I, the
// isolated vertices of the inverse graph) are taken in closed form -- a node
// (S', C, l') contributes the C(|I|, l') ways to finish S' from I -- and the
// branching runs on the rest: the child of v_i in C (in order) keeps the
// vertices of C after v_i that are adjacent to v_i (Eq. kCtPlex: C minus v_1..
// v_i minus v_i's neighbours in the inverse graph), l' - 1, when it still
// holds enough vertices with I.  Children with l' - 1 <= 1 are counted at
// once (l' - 1 = 1: |I| + |C_i|; 0: one clique).  Frames (C, l', last v)
// live in the child-queue area of LDS: depth <= l <= KCT_MAX_L.
constexpr int KCT_MAX_L = 96;

template <int W>
struct KctFrame {
    uint64_t C[W];
    int32_t l, cur;
};
static_assert(sizeof(KctFrame<4>) * KCT_MAX_L <= 2 * QCAP * sizeof(int32_t) &&
                  sizeof(KctFrame<1>) * KCT_MAX_L <= 2 * 260 * sizeof(int32_t),
              "kCtPlex frames must fit the queue area");

template <int W>
__device__ u128 tplex_branch_count(SearchMem<W>& M, const uint64_t (&P)[W], int pc, int l, bool& ovf,
                                   uint64_t& nodes) {
    const int lane = lane_id();
    // I: vertices of P adjacent to all others of P
    uint64_t I[W];
#pragma unroll
    for (int q = 0; q < W; ++q) {
        bool full = false;
        if ((P[q] >> lane) & 1) {
            int d = 0;
#pragma unroll
            for (int w = 0; w < W; ++w) d += popc64(P[w] & M.rows[lane + 64 * q][w]);
            full = d == pc - 1;
        }
        I[q] = uni64(ballot(full));
    }
    const int nI = popcW(I);
    auto add = [&](u128& acc, u128 x) {
        acc += x;
        ovf |= acc < x;
    };
    KctFrame<W>* fr = reinterpret_cast<KctFrame<W>*>(&M.pq[0][0]);
    u128 total = 0;
    add(total, binom128(nI, l, ovf));  // the root: all l vertices from I
    int sp = 0;
    if (lane == 0) {
#pragma unroll
        for (int w = 0; w < W; ++w) fr[0].C[w] = P[w] & ~I[w];
        fr[0].l = l;
        fr[0].cur = -1;
    }
    wave_sync();
    while (sp >= 0) {
        uint64_t C[W];
#pragma unroll
        for (int w = 0; w < W; ++w) C[w] = uni64(fr[sp].C[w]);
        const int lf = uniform_i32(fr[sp].l), cur = uniform_i32(fr[sp].cur);
        int v = -1;  // next vertex of C after cur
#pragma unroll
        for (int w = W - 1; w >= 0; --w) {
            const uint64_t b = C[w] & (cur < 0 ? ~0ull : upper_mask(cur, w));
            if (b) v = 64 * w + __builtin_ctzll(b);
        }
        if (v < 0) {
            --sp;
            continue;
        }
        if (lane == 0) fr[sp].cur = v;
        const int lc = lf - 1;
        ++nodes;
        if (lc == 0) {
            add(total, 1);
            wave_sync();
            continue;
        }
        uint64_t Ci[W];
#pragma unroll
        for (int w = 0; w < W; ++w) Ci[w] = C[w] & M.rows[v][w] & upper_mask(v, w);
        const int ci = popcW(Ci);
        if (ci + nI < lc) {
            wave_sync();
            continue;
        }
        if (lc == 1) {  // C(|I|, 1) from I, and each vertex of C_i
            add(total, (u128)(nI + ci));
            wave_sync();
            continue;
        }
        add(total, binom128(nI, lc, ovf));  // the child: the rest from I
        if (lane == 0) {
#pragma unroll
            for (int w = 0; w < W; ++w) fr[sp + 1].C[w] = Ci[w];
            fr[sp + 1].l = lc;
            fr[sp + 1].cur = -1;
        }
        ++sp;
        wave_sync();
    }
    wave_sync();
    return total;
}

}  // namespace

// The build's work areas alias the search's per-vertex scratch, child queue
// and LDS frames (md .. fr), which the search writes before it reads.
template <int W>
constexpr bool build_fits() {
    return build_scratch_bytes<W>() <= (int)(sizeof(SearchMem<W>) - offsetof(SearchMem<W>, md));
}
static_assert(build_fits<1>() && build_fits<2>() && build_fits<3>() && build_fits<4>(),
              "sub-branch build scratch must fit the search's LDS");

// ---------------------------------------------------------------- split queue
// The counters and the items are accessed relaxed at device scope, and order
// comes from waiting (device_util.h): a wave's reservation has returned before
// the wave can stop counting as working, and a wave that has read that no wave
// works reads the reservations after it, so it sees every item pushed before
// the last one stopped; an item's fields are done before its ready flag is set,
// and read after it.  (Sequentially consistent counters and a released flag
// wrote back and dropped whole caches several times an item.)
//
// The loads of the waiting waves queue up with the counters' updates: with all
// 4,096 waves of a launch waiting, an item cost some 13 us of the launch, one
// after the other and whatever it held.  So at most SQ_WAITERS waves wait, and
// the longer one has waited the longer it naps, up to a sixteenth of its wait
// (which the end of the launch may be noticed later) or 256 sleeps, 0.5 ms.
// R-MAT s13 at k = 32 and 35 (733,122 and 14,193 nodes) 381 and 21.3 ms before,
// 24.9 and 2.5 now; G(300, 0.6) at k = 12 136 and 59 ms.  512 waiting waves:
// 20.9, 1.8 and 57 ms, but a quarter of the device's waves should be at hand
// where a few roots hold most of the work.  Without the limit, with the naps
// 41.9, 6.6 and 63 ms; with the limit of 512 alone 21.3, 1.7 and 74 ms.
constexpr unsigned long long SQ_WAITERS = 1024;
constexpr uint64_t SQ_NAP_TICKS = 3200;  // sixteen sleeps of about 2 us, in ticks of the 100 MHz clock
constexpr int SQ_POLL_BUSY = 256, SQ_POLL_HUNGRY = 4;
constexpr uint64_t SQ_POLL_TICKS = 2000;  // 20 us of the 100 MHz clock
// longest time a wave waits while the queue shows no progress (no item
// claimed or reserved, no change in the working waves) before it gives up
// with ERR_QUEUE (constant-rate clock of 100 MHz: 60 s); also at most
// SQ_WAIT_SPINS sleeps (each at least 64 * 32 clocks), so the wait ends even
// if that clock did not advance
constexpr uint64_t SQ_WAIT_TICKS = 6000000000ull;
constexpr uint64_t SQ_WAIT_SPINS = 1ull << 26;

__device__ __forceinline__ void sq_add(unsigned long long* p, long long v) { (void)dev_add(p, (unsigned long long)v); }
// No wave works and no item waits, read in this order.
__device__ __forceinline__ bool nothing_left(unsigned long long* sq) {
    if (dev_load(&sq[SQ_BUSY]) != 0) return false;
    wait_memory();
    const unsigned long long r = dev_load(&sq[SQ_RESERVE]);
    return dev_load(&sq[SQ_HEAD]) >= r;
}

// An idle wave claims a queued node: returns its index once its producer has
// written it, or -1 when no wave is working and the queue is empty (then no
// item can appear any more: an item is pushed only by a working wave, before
// that wave stops counting as working) or after SQ_WAIT_TICKS without work
// (ERR_QUEUE).  A claim takes the head first and counts the wave as working
// after it; a wave in between may process that node while others have
// finished, and handles whatever it pushes itself.  Idle polling backs off.
__device__ int64_t queue_take(const SearchArgs& a) {
    unsigned long long* sq = a.sq;
    uint64_t t0 = wall_clock64();
    const uint64_t t_in = t0;
    unsigned long long seen_h = ~0ull, seen_r = ~0ull, seen_b = ~0ull;
    int nap = 1;
    for (uint64_t spin = 0;; ++spin) {
        long long got = -1;
        int done = 0;
        if (lane_id() == 0) {
            const unsigned long long h = dev_load(&sq[SQ_HEAD]), r = dev_load(&sq[SQ_RESERVE]);
            const unsigned long long bz = dev_load(&sq[SQ_BUSY]);
            if (h != seen_h || r != seen_r || bz != seen_b) {  // progress: the wait starts again
                seen_h = h;
                seen_r = r;
                seen_b = bz;
                t0 = wall_clock64();
                spin = 0;
            }
            if (h < r && atomicCAS(&sq[SQ_HEAD], h, h + 1) == h) {
                got = (long long)h;
                sq_add(&sq[SQ_BUSY], 1);
                sq_add(&sq[SQ_IDLE], -1);
            } else if (h >= r && bz == 0 && nothing_left(sq)) {
                done = 1;
            } else if (wall_clock64() - t0 > SQ_WAIT_TICKS || spin > SQ_WAIT_SPINS) {
                atomicOr(a.err, ERR_QUEUE);
                done = 1;
            }
            if (got >= 0) {  // the producer reserved the slot before writing it
                for (uint64_t wspin = 0; dev_load(&a.squeue[got].ready) == 0; ++wspin) {
                    if (wall_clock64() - t0 > SQ_WAIT_TICKS || wspin > SQ_WAIT_SPINS) {
                        atomicOr(a.err, ERR_QUEUE);
                        got = -1;
                        done = 1;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(2);
                }
            }
        }
        got = (long long)uni64((uint64_t)__shfl(got, 0, 64));
        done = uniform_i32(__shfl(done, 0, 64));
        if (got >= 0) {
            wait_memory();  // the flag was read before the fields are
            return got;
        }
        if (done) return -1;
        for (int i = 0; i < nap; ++i) __builtin_amdgcn_s_sleep(64);
        const uint64_t most = (wall_clock64() - t_in) / SQ_NAP_TICKS;
        nap = nap < 32 ? 2 * nap : (most > 256 ? 256 : (most > 32 ? (int)most : 32));
    }
}

// BUILD = false: each task's g_i is loaded from the arena.  BUILD = true
// (batches too large for arenas): the task's slot is its seed edge id in
// graph task_graph[i], and the wave builds g_i in LDS first (build.h).
// DEEP = false: tasks with l <= 5 at the root (k <= 7), which never branch:
// a root is finished in closed form or its children are counted by lanes.
// Without frames, the split queue, 128-bit sums and the 3- and t-plex forms
// the kernel is a third of the size (the instruction cache holds 64 KB for two
// compute units) and keeps more in registers (the one-word class 105 without
// spills): k = 5, 6, 7 on R-MAT s18 6.0, 14.0, 161 ms against 4.1, 12.1, 152 ms.
template <int W, bool BUILD, bool DEEP>
__global__ __launch_bounds__(256, (W <= 2 ? 4 : (W <= 3 ? 3 : 2))) void k_search(SearchArgs a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    SearchMem<W>& M = reinterpret_cast<SearchMem<W>*>(smem_raw)[threadIdx.x / 64];
    Frame<W>* gfr = DEEP && a.gframes ? reinterpret_cast<Frame<W>*>(a.gframes) +
                                    ((int64_t)blockIdx.x * 4 + threadIdx.x / 64) * GLOBAL_FRAMES
                              : nullptr;
    // frames past the LDS ones live in this wave's slab of device memory;
    // every lane writes them (identical values) and reads back its own stores
    auto FR = [&](int d) -> Frame<W>& { return d < LDS_FRAMES ? M.fr[d] : gfr[d - LDS_FRAMES]; };
    const int lane = lane_id();
    const int opts = a.opts;
    const bool rule1 = opts & OPT_RULE1, rule2 = opts & OPT_RULE2, et = opts & OPT_ET;
    const bool work = opts & OPT_WORK;
    Acc acc{0, false};
    uint64_t wk_tasks = 0, wk_nodes = 0, wk_ops = 0;
    const uint64_t t_wave0 = work ? wall_clock64() : 0;
    // runtime splitting: a wave counts as working from its start until the
    // static tasks run out, then takes queued nodes until none is left
    const bool splitting = DEEP && a.squeue != nullptr;
    if (splitting && lane == 0) {
        sq_add(&a.sq[SQ_BUSY], 1);
        M.pushed = 0;
    }
    bool on_queue = false, took_item = false;
    int poll_in = 0;      // candidate nodes until the queue counters are read again
    uint64_t poll_t = 0;  // when they were read last
    bool hungry = false;  // some wave waited for work at the last reading
    // lane j: the least |P| with C(|P|, j) >= split_bound (a node with l = j
    // and fewer candidates is never handed over), so that the test per node
    // is a lane read instead of a table load
    int push_pmin = 1 << 20;
    if (splitting) {
        const int j = lane;
        int lo = j > 0 ? j : 1, hi = 64 * MAX_W + 1;  // C(hi, j) may stay below the bound: then never
        if (j > 0 && binom(hi, j) >= a.split_bound) {
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (binom(mid, j) >= a.split_bound) hi = mid; else lo = mid + 1;
            }
            push_pmin = lo;
        }
    }

    Drawn drawn;
    for (;;) {
        int64_t it = 0;
        int64_t qitem = -1;
        if (!on_queue) {
            it = drawn.next(a.tickets);
            if (it < 0) {
                if (!splitting) break;
                on_queue = true;
                int stay = 1;
                if (lane == 0) {
                    // waiting waves enough: this one ends, unless it handed nodes
                    // over (whoever did stays until the queue is empty)
                    stay = dev_add(&a.sq[SQ_IDLE], 1ull) < SQ_WAITERS || M.pushed;
                    if (!stay) sq_add(&a.sq[SQ_IDLE], -1);
                    sq_add(&a.sq[SQ_BUSY], -1);
                }
                if (!uniform_i32(stay)) break;
            }
        }
        if (on_queue) {
            if (took_item && lane == 0) {  // the last queued node is done (its pushes are visible)
                sq_add(&a.sq[SQ_IDLE], 1);
                sq_add(&a.sq[SQ_BUSY], -1);
            }
            qitem = queue_take(a);
            if (qitem < 0) break;
            took_item = true;
            it = (int64_t)uni64((uint64_t)dev_load(&a.squeue[qitem].it));
        }
        const bool listed = it < a.nexplicit;
        const int64_t task = listed ? a.tasks[it] : 0;
        const int64_t slot = listed ? task_slot(task) : (int64_t)a.slots[it - a.nexplicit];
        // A range [sx, x1) of root vertices only ever uses the vertices from sx
        // on (a clique's first vertex is its lowest), so it is searched as
        // [0, x1 - sx) of the sub-branch on those: fewer words a row, and the
        // range may belong to a narrower class than its slot (R-MAT s18 at
        // k = 7 161 ms and k = 8 3.83 s, against 180 ms and 4.78 s with every
        // range on its slot's width).  A queued node is a whole node below the
        // root: every first vertex.
        const int sx = listed && !BUILD ? task_x0(task) : 0;
        const int x1 = !listed || qitem >= 0 ? 64 * W : task_x1(task) - sx;
        const int gi = a.task_graph ? uniform_i32(a.task_graph[it]) : 0;
        const int k = a.graph_k ? uniform_i32(a.graph_k[gi]) : a.k;
        int c = 0, words = W;  // vertices used; words a row of the slot has
        int64_t ro = 0, vo = 0;
        if constexpr (BUILD) {
            c = uniform_i32(a.bviews[gi].subsize[slot]);
        } else {
            const ArenaView& A = a.views ? a.views[gi] : a.A;
            c = uniform_i32(A.seed_c[slot]);
            words = (c + 63) >> 6;
            c -= sx;
            ro = A.row_off[slot] + (int64_t)sx * words;
            vo = A.vtx_off[slot] + sx;
        }
        // t of the closed forms: fixed, or 2 when 2k <= tau and 3 above (Section 6.1)
        const int tau_g = a.graph_tau ? uniform_i32(a.graph_tau[gi]) : a.tau;
        const int tpl = a.tplex > 0 ? a.tplex : (2 * k <= tau_g ? 2 : 3);
        const bool t2 = et && tpl >= 2, t3 = et && tpl >= 3, t4 = et && tpl >= 4;
        wk_tasks += work;
        std::conditional_t<DEEP, Acc, Acc64> tacc{0, false};
        if (k == 3) {  // l = 1 at the root: |V(g_i)| triangles through the seed edge
            tacc.add((uint64_t)c);
            goto task_done;
        }

        if constexpr (BUILD) {
            // ---- build g_i in LDS, vertices in colour order (build.h)
            const BuildGraph& B = a.bviews[gi];
            const BuildScratch<W> S = BuildScratch<W>::carve(&M.md[0]);
            const int32_t e = (int32_t)slot;
            uint32_t twoE = 0;
            // l = 2 at the root needs the edges' number alone; a search without
            // branching takes sparse sub-branches in candidate order, every vertex
            // its own colour (any order and proper colouring give the same count;
            // colouring and reordering 40 vertices is half of a task's instructions).
            // With the prefixes found by the wave and the folded pairs of build.h:
            // ten graphs of up to 5,000 vertices 65 -> 43 ms
            const int plain = DEEP ? PLAIN_NEVER : (k == 4 ? PLAIN_ALWAYS : PLAIN_SPARSE);
            if (build_subbranch<W>(B.G, B.G.eu[e], B.G.ev[e], B.G.rank[e], c, nullptr, B.vcol, M.rows, M.col, S, &twoE,
                                   plain) < 0) {
                if (lane == 0) atomicOr(a.err, ERR_WIDTH);
                goto task_done;
            }
            if (!DEEP && k == 4) {
                tacc.add((uint64_t)(twoE / 2));
                goto task_done;
            }
            if (!DEEP && plain_build(plain, c, twoE)) {
                for (int i = lane; i < c; i += 64) M.col[i] = (int16_t)(c - i);
                wave_sync();
            } else {
            int npos[W];
            order_positions<W>(c, M.col, S, npos);
            uint64_t nr[W][W];
            int16_t nc[W];
#pragma unroll
            for (int q = 0; q < W; ++q) {
                const int i = lane + 64 * q;
                nc[q] = 0;
                if (i < c) {
                    relabelled_row<W>(M.rows, i, S, nr[q]);
                    nc[q] = M.col[i];
                }
            }
            wave_sync();
#pragma unroll
            for (int q = 0; q < W; ++q) {
                if (lane + 64 * q < c) {
#pragma unroll
                    for (int w = 0; w < W; ++w) M.rows[npos[q]][w] = nr[q][w];
                    M.col[npos[q]] = nc[q];
                }
            }
            wave_sync();
            }
        } else {
            // ---- load the sub-branch into LDS (coalesced)
            const ArenaView& A = a.views ? a.views[gi] : a.A;
            if (sx == 0 && words == W) {
                for (int i = lane; i < c * W; i += 64) (&M.rows[0][0])[i] = A.rows[ro + i];
            } else {  // rows sx .. without their first sx bits
                const int s = sx >> 6, b = sx & 63;
                for (int i = lane; i < c * W; i += 64) {
                    const int v = i / W, w = i - v * W + s;
                    const uint64_t* src = A.rows + ro + (int64_t)v * words;
                    uint64_t x = w < words ? src[w] >> b : 0;
                    if (b && w + 1 < words) x |= src[w + 1] << (64 - b);
                    (&M.rows[0][0])[i] = x;
                }
            }
            for (int i = lane; i < c; i += 64) M.col[i] = A.col[vo + i];
            wave_sync();
        }
        {
        // W = 1: lane v keeps vertex v's later neighbours, and the leaves' counts
        // and queued children are kept over the whole task (they all refer to
        // the same rows), so that a node pays no reduction and the lanes count
        // children of many nodes at once.  A set of at most 64 vertices adds at
        // most 2^25 to a lane's leaf_S (each of its terms below is under 6
        // million) and 2^22 to leaf_usum, a child under 2^16 to leaf_sum, so
        // 64-bit sums over the lanes hold 2^32 sets: over an hour of one wave at
        // a microsecond a set
        uint64_t dagv = 0, leaf_sum = 0, leaf_usum = 0;
        int64_t leaf_S = 0;
        int q1 = 0, q1_lc = 0;
        if constexpr (W == 1) {
            dagv = lane < c ? M.rows[lane][0] & upper_mask(lane, 0) : 0;
            M.dag[lane] = dagv;
            wave_sync();
        }
        // colour class lane + 64 q (colour lane + 64 q + 1) occupies the
        // relabelled positions [cs0[q], cs1[q]) = [#(col > colour), #(col >= colour))
        int cs0[W], cs1[W];
        const int ncol = uniform_i32(M.col[0]);
        const int ncq = (ncol + 63) >> 6;
#pragma unroll
        for (int q = 0; q < W; ++q) {
            const int cv = lane + 64 * q + 1;
            int lo = 0, hi = c;
            while (lo < hi) { int mid = (lo + hi) >> 1; if (M.col[mid] > cv) lo = mid + 1; else hi = mid; }
            const int s0 = lo;
            hi = c;
            while (lo < hi) { int mid = (lo + hi) >> 1; if (M.col[mid] >= cv) lo = mid + 1; else hi = mid; }
            cs0[q] = s0;
            cs1[q] = cv <= ncol ? lo : s0;
        }

        // W = 1: count the queued children, one per lane: edges inside Q (l = 2)
        // or triangles (l = 3, the queue first sorted by |Q| >> 3 in ballot
        // passes, since a lane's work grows with |Q|; bit 0 of an entry, never a
        // member, says that its parent was dense)
        auto drain1 = [&]() __attribute__((always_inline)) {
            if constexpr (W == 1) {
                if (q1 == 0) return;
                wave_sync();
                int cur = 0;
                if (q1_lc == 3 && q1 > 64) {
                    for (int b = 3; b < 6; ++b) {
                        const uint64_t* src = M.q1[cur];
                        uint64_t* dst = M.q1[cur ^ 1];
                        int nz = 0;
                        for (int i0 = 0; i0 < q1; i0 += 64) {
                            const int i = i0 + lane;
                            nz += popc64(ballot(i < q1 && !((popc64(src[i]) >> b) & 1)));
                        }
                        int z0 = 0, o0 = nz;
                        for (int i0 = 0; i0 < q1; i0 += 64) {
                            const int i = i0 + lane;
                            const bool valid = i < q1;
                            const uint64_t e = valid ? src[i] : 0;
                            const bool one = valid && ((popc64(e) >> b) & 1);
                            const uint64_t bo = ballot(one), bz = ballot(valid && !one);
                            if (valid) dst[one ? o0 + popc64(bo & lanemask_lt()) : z0 + popc64(bz & lanemask_lt())] = e;
                            z0 += popc64(bz);
                            o0 += popc64(bo);
                        }
                        wave_sync();
                        cur ^= 1;
                    }
                }
                uint64_t lops = 0;
                for (int i0 = 0; i0 < q1; i0 += 64) {
                    if (i0 + lane < q1) {
                        const uint64_t e = M.q1[cur][i0 + lane];
                        if (q1_lc == 3) {
                            const uint64_t Q[1] = {e & ~1ull};
                            leaf_sum += lane_triangles<1>(reinterpret_cast<const uint64_t(*)[1]>(M.rows), Q, e & 1, lops);
                        } else {
                            leaf_sum += lane_edges1(M.dag, e & ~1ull);
                        }
                    }
                }
                if (work) wk_ops += uni64(wave_sum(lops));
                q1 = 0;
                wave_sync();
            }
        };

        // Count a node that needs no branching: returns true and sets val, or
        // false when the node (l >= 4) must be branched on.
        using val_t = std::conditional_t<DEEP, u128, uint64_t>;
        auto choose = [&](int n, int r) -> val_t {
            if constexpr (DEEP) return binom128(n, r, tacc.ovf);
            else return binom(n, r);
        };
        auto finish = [&](const uint64_t (&P)[W], int l, val_t& val) -> bool {
            const int pc = popcW(P);
            val = 0;
            if (work) { wk_nodes += 1; wk_ops += W; }
            if (pc < l) return true;
            if (l == 1) { val = (uint64_t)pc; return true; }
            int mn = 1 << 30, nf = 0;
            uint32_t dsum = 0, s2 = 0;
#pragma unroll
            for (int q = 0; q < W; ++q) {
                if ((P[q] >> lane) & 1) {
                    int d = 0;
#pragma unroll
                    for (int w = 0; w < W; ++w) d += popc64(P[w] & M.rows[lane + 64 * q][w]);
                    mn = d < mn ? d : mn;
                    nf += (d == pc - 1);
                    dsum += d;
                    const int cm = pc - 1 - d;
                    s2 += (uint32_t)(cm * (cm - 1) / 2);
                }
            }
            if (work) wk_ops += (uint64_t)pc * W;
            const uint64_t twoE = wsum_u32(dsum);
            if (l == 2) { val = twoE / 2; return true; }
            if (et) {
                const int mind = wmin_i32(mn);
                if (mind >= pc - 1) { val = choose(pc, l); return true; }
                if (t2 && mind >= pc - 2) {
                    const int nfull = (int)wsum_u32((uint32_t)nf);
                    if constexpr (DEEP) val = twoplex_count(nfull, (pc - nfull) / 2, l, tacc.ovf);
                    else val = twoplex_small(nfull, (pc - nfull) / 2, l);
                    return true;
                }
                if (l == pc) { val = 0; return true; }  // P itself is not a clique
                if constexpr (DEEP) {
                    const bool plex3 = t3 && mind >= pc - 3, plext = t4 && mind >= pc - tpl && l <= KCT_MAX_L;
                    if (plex3) {
                        val = threeplex_count<W>(M, P, pc, l, tacc.ovf);
                        return true;
                    }
                    if (plext) {
                        uint64_t kn = 0;
                        val = tplex_branch_count<W>(M, P, pc, l, tacc.ovf, kn);
                        if (work) { wk_nodes += kn; wk_ops += kn * W; }
                        return true;
                    }
                }
            }
            if (l != 3) return false;
            // triangles inside P: dense -> missing-pair identity, sparse -> DAG edges
            const uint64_t p64 = (uint64_t)pc;
            const uint64_t Mp = (p64 * (p64 - 1) - twoE) / 2;
            uint32_t t = 0;
            const bool dense = Mp <= twoE / 2;
#pragma unroll
            for (int q = 0; q < W; ++q) {
                const int z = lane + 64 * q;
                if ((P[q] >> lane) & 1) {
                    uint64_t Cz[W];
#pragma unroll
                    for (int w = 0; w < W; ++w)
                        Cz[w] = P[w] & (dense ? ~M.rows[z][w] : M.rows[z][w]) & upper_mask(z, w);
#pragma unroll
                    for (int wy = 0; wy < W; ++wy) {
                        while (Cz[wy]) {
                            const int y = wy * 64 + __builtin_ctzll(Cz[wy]);
                            Cz[wy] &= Cz[wy] - 1;
#pragma unroll
                            for (int w = 0; w < W; ++w) {
                                const uint64_t row = dense ? ~M.rows[y][w] : M.rows[y][w];
                                if (w >= wy) t += popc64(Cz[w] & row);
                            }
                        }
                    }
                }
            }
            if (work) wk_ops += (dense ? Mp : twoE / 2) * W;
            const uint64_t T = wsum_u32(t);
            if (dense) {
                const uint64_t S2 = wsum_u32(s2);
                val = p64 * (p64 - 1) * (p64 - 2) / 6 - Mp * (p64 - 2) + S2 - T;
            } else {
                val = T;
            }
            return true;
        };

        // 4-cliques inside R (r >= 4 vertices) from the missing pairs H of R:
        // inclusion-exclusion over the edge sets of H spanning at most four
        // vertices gives K4 = C(r,4) - M C(r-2,2) + P3 (r-3) + 2K2 - T (r-3)
        // - P4 - S3 + C4 + paw - diamond + K4(H), with P3 the 2-paths, 2K2
        // the disjoint pairs, T the triangles, P4 the 3-paths, S3 the 3-stars,
        // C4 the 4-cycles, paw, diamond and K4(H) the remaining 4-vertex
        // shapes of H.  All but C(r,4) + C(M,2) is a sum over the vertices,
        // missing pairs and 2-paths of H, taken by the lanes holding them
        // into S (24 times its value, so that every term is an integer).
        // Returns false, counting nothing, when H is too dense for this to
        // beat branching on the pairs of R.  (Spreading all pairs of R over
        // the lanes instead evens out vertices with many missing pairs, but
        // costs ~r^2 / 64 rounds even for a nearly complete R; on R-MAT s18
        // at k = 9 it made the search 1.7x slower.)
        auto k4_missing = [&](auto wv, const auto& R, auto rows, int r, bool whole, int64_t& S, uint64_t& uacc,
                              bool& rdense) -> bool {
            constexpr int WV = decltype(wv)::value;
            // the vertices of R, packed onto consecutive lanes
            {
                int base = 0;
#pragma unroll
                for (int q = 0; q < WV; ++q) {
                    if ((R[q] >> lane) & 1) M.vl[base + popc64(R[q] & lanemask_lt())] = (int16_t)(lane + 64 * q);
                    base += popc64(R[q]);
                }
            }
            wave_sync();
            const int rounds = (r + 63) >> 6;
            int msum = 0;
            for (int t = 0; t < rounds; ++t) {
                const int j = 64 * t + lane;
                if (j < r) {
                    const int v = M.vl[j];
                    int mv = -1;  // R & ~row(v) holds v itself
#pragma unroll
                    for (int w = 0; w < WV; ++w) mv += popc64(R[w] & ~rows[v][w]);
                    M.md[v] = (int16_t)mv;
                    msum += mv;
                }
            }
            const int Msum = (int)wsum_u32((uint32_t)msum);
            // The lanes run in lockstep, so this evaluation takes as long as
            // its busiest lane: ~18 instructions for each missing pair it
            // holds (half of those at its vertices) and ~12 for each triangle
            // of missing pairs there (about its pairs' pairs times the density
            // of H), plus ~150 for the reductions and ~12 for each tile of the
            // codegrees.  Weights of 50 / 100 / 200 / 500 % of the estimate: R-MAT
            // s14 k = 8 17.4 / 17.5 / 17.9 / 20.0 ms, s16 222 / 223 / 228 / 257,
            // G(250, .8) 71.7 / 74.9 / 80.9 / 99.0; never 42.7, 999 and 285.
            // The alternative for one R = P & N+(x) of an l = 5 node is one
            // child y per lane counting the triangles of R & N+(y): ~35
            // instructions per vertex of the largest child, ~ r * d, per 64
            // children (r of them here, sharing rounds with the other x
            // through the queue); for a whole l = 4 node it is that for every
            // x (~18 instructions a step), ~ |E(R)| * d / 64 rounds of 64
            // children.
            const float lmax = (float)wmax_i32(msum);
            const float pairs = 0.5f * (float)r * (float)(r - 1);
            const float E = pairs - 0.5f * (float)Msum, d = E / pairs;
            rdense = 2.0f * E >= pairs;
            const int nb = (r + 15) >> 4;
            const float cost = a.k4_weight * (9.0f * lmax + 3.0f * lmax * lmax * (1.0f - d) / (float)rounds + 150.0f +
                                              6.0f * (float)(nb * (nb + 1)));
            const float alt = whole ? 18.0f * E * d * (float)r * d / 64.0f
                                    : 35.0f * (float)r * d * (float)r / 64.0f;
            if (!(a.k4_weight > 0.f) || cost > alt) return false;
            if (work) wk_ops += (uint64_t)(r + Msum) * WV;
            const int64_t Mh = Msum / 2;
            const uint64_t r64 = (uint64_t)r;
            uacc += r64 * (r64 - 1) * (r64 - 2) * (r64 - 3) / 24 + (uint64_t)(Mh * (Mh - 1) / 2);
            if (Msum == 0) return true;
            wave_sync();  // md[] of every vertex of R
            const int64_t c2 = (int64_t)(r - 2) * (r - 3) / 2;
            for (int t = 0; t < rounds; ++t) {
                const int j = 64 * t + lane;
                if (j >= r) continue;
                const int v = M.vl[j];
                const int64_t mv = M.md[v];
                S += -12 * c2 * mv + 24 * (int64_t)(r - 4) * (mv * (mv - 1) / 2) - 4 * mv * (mv - 1) * (mv - 2) -
                     3 * (2 * mv * mv + 5 * mv + 1);  // the last: the codegrees' part, below
                if (mv == 0) continue;
                uint64_t hv[WV];
#pragma unroll
                for (int w = 0; w < WV; ++w)
                    hv[w] = R[w] & ~rows[v][w] & (w == (v >> 6) ? ~(1ull << (v & 63)) : ~0ull);
                // missing pairs v-u, each taken at one end: at the smaller when
                // v and u have the same parity, else at the larger, so that a
                // vertex holds about half of its pairs wherever it lies.
                // Codegree cc in H (triangles, diamonds, paws), the 3-paths
                // through v-u, K4(H).  Per-v sums in 32 bits: a1 = sum cc,
                // a2 = sum cc (m_u - cc), a3 = sum (m_u - 1)
                const uint64_t par = (v & 1) ? 0xAAAAAAAAAAAAAAAAull : 0x5555555555555555ull;
                int32_t a1 = 0, a2 = 0, a3 = 0;
#pragma unroll
                for (int wu = 0; wu < WV; ++wu) {
                    uint64_t bu = hv[wu] & ~(upper_mask(v, wu) ^ par);
                    while (bu) {
                        const int u = wu * 64 + __builtin_ctzll(bu);
                        bu &= bu - 1;
                        uint64_t X[WV];
                        int cc = -1;  // u lies in both hv and R & ~row(u)
#pragma unroll
                        for (int w = 0; w < WV; ++w) {
                            X[w] = hv[w] & ~rows[u][w];
                            cc += popc64(X[w]);
                        }
                        const int mu = M.md[u];
                        a1 += cc;
                        a2 += cc * (mu - cc);
                        a3 += mu - 1;
                        if (cc >= 2) {
                            const int top = u > v ? u : v;
#pragma unroll
                            for (int w = 0; w < WV; ++w) X[w] &= upper_mask(top, w);
#pragma unroll
                            for (int wx = 0; wx < WV; ++wx) {
                                while (X[wx]) {
                                    const int z = wx * 64 + __builtin_ctzll(X[wx]);
                                    X[wx] &= X[wx] - 1;
                                    int kk = 0;
#pragma unroll
                                    for (int w = 0; w < WV; ++w)
                                        if (w >= wx) kk += popc64(X[w] & ~rows[z][w]);
                                    S += 24 * kk;
                                }
                            }
                        }
                    }
                }
                // per missing pair, doubled: 24 (cc - (m_u-1)(m_v-1)) - 8 (r-3) cc - 12 cc (cc-1) for the
                // triangles, 3-paths and diamonds, 12 cc (m_u + m_v - 4) for the paws, -24 cc below
                S += (int64_t)(12 * (mv - 4) - 8 * (r - 3) + 12) * a1 + 12 * (int64_t)a2 - 24 * (mv - 1) * (int64_t)a3;
            }
            // 2-paths a-v-b: 4 C4 = Z = sum over a < b of codeg (codeg - 1); 2 Z
            // is the sum over a != b of codeg^2 less that of codeg, the latter
            // sum_v m_v (m_v - 1).  With self pairs in H an entry is codeg plus
            // 2 on missing pairs, the diagonal m + 1, so the sum of all squares
            // exceeds that of codeg^2 by 4 (2 sum_pairs cc) + 4 sum m + sum
            // (m + 1)^2.  C4 enters
            // with 24 Z / 4 = 3 (2 Z):
            S += 3 * (int64_t)codegree_squares<WV, WV <= 2 && !DEEP ? 4 : 2>(R, rows, M.vl, r);
            return true;
        };

        // children of a node with l = 5 (l = 4), x below xhi: the
        // 4-cliques (triangles) of R = P & N+(x) for each x.  A dense R is
        // counted by the wave from its missing pairs; otherwise its children
        // (x, y) join a queue in LDS and every 64 queued children are counted
        // one per lane.
        auto children_by_lanes = [&](auto wv, const auto& P, auto rows, const int16_t* col, int cn, int l, int xhi) {
            constexpr int WV = decltype(wv)::value;
            uint64_t lsum = 0, lops = 0, usum = 0;
            int64_t S = 0;
            const int lc = l - 2;
            int qn = 0;
            // Count the queued children [base, base + cnt), cnt <= 64, one per lane.
            auto run_queue = [&](const int32_t* q, int base, int cnt) {
                if (lane < cnt) {
                    const int e = q[base + lane];
                    const int x = (e >> 8) & 0xFF, y = e & 0xFF;
                    uint64_t Q[WV];
#pragma unroll
                    for (int w = 0; w < WV; ++w) Q[w] = P[w] & rows[x][w] & rows[y][w] & upper_mask(y, w);
                    if (lc == 3) lsum += lane_triangles<WV>(rows, Q, (e >> 25) & 1, lops);
                    else lsum += lane_edges<WV>(rows, Q);
                }
            };
            // Count every queued child: a lane's work grows with |Q|, so the
            // queue is first sorted by |Q| (stable LSD passes over |Q| >> 3,
            // ballot partitions) and counted 64 at a time in that order.
            auto drain = [&]() {
                wave_sync();
                int cur = 0;
                if (qn > 64) {
                    for (int b = 19; b < 24; ++b) {
                        const int32_t* src = M.pq[cur];
                        int32_t* dst = M.pq[cur ^ 1];
                        int nz = 0;
                        for (int i0 = 0; i0 < qn; i0 += 64) {
                            const int i = i0 + lane;
                            nz += popc64(ballot(i < qn && !((src[i] >> b) & 1)));
                        }
                        int z0 = 0, o0 = nz;
                        for (int i0 = 0; i0 < qn; i0 += 64) {
                            const int i = i0 + lane;
                            const bool valid = i < qn;
                            const int e = valid ? src[i] : 0;
                            const bool one = valid && ((e >> b) & 1);
                            const uint64_t bo = ballot(one), bz = ballot(valid && !one);
                            if (valid) dst[one ? o0 + popc64(bo & lanemask_lt()) : z0 + popc64(bz & lanemask_lt())] = e;
                            z0 += popc64(bz);
                            o0 += popc64(bo);
                        }
                        wave_sync();
                        cur ^= 1;
                    }
                }
                for (int i0 = 0; i0 < qn; i0 += 64) run_queue(M.pq[cur], i0, qn - i0 < 64 ? qn - i0 : 64);
                qn = 0;
                wave_sync();
            };
            bool done = false;
            if (l == 4 && xhi >= cn) {
                const int pc = popcW(P);
                bool pd = false;
                done = pc < 4 || k4_missing(wv, P, rows, pc, true, S, usum, pd);
            }
            int xx = -1;
            while (!done) {
                int nx = -1;
#pragma unroll
                for (int w = WV - 1; w >= 0; --w) {
                    const uint64_t b = P[w] & (xx < 0 ? ~0ull : upper_mask(xx, w));
                    if (b) nx = w * 64 + __builtin_ctzll(b);
                }
                if (nx < 0 || nx >= xhi || (rule1 && col[nx] < l)) break;
                xx = nx;
                uint64_t Rx[WV];
#pragma unroll
                for (int w = 0; w < WV; ++w) Rx[w] = uni64(P[w] & rows[xx][w] & upper_mask(xx, w));
                const int rc = popcW(Rx);
                if (rc < lc + 1) continue;
                if (work) { wk_nodes += rc; wk_ops += (uint64_t)rc * WV; }
                bool rdense = false;
                if (l == 5 && k4_missing(wv, Rx, rows, rc, false, S, usum, rdense)) continue;
#pragma unroll
                for (int q = 0; q < WV; ++q) {
                    const int y = 64 * q + lane;
                    const bool act = ((Rx[q] >> lane) & 1) && !(rule1 && col[y] < l - 1);
                    const uint64_t bq = ballot(act);
                    if (act) {
                        int qy = 0;  // |Q| of the child (x, y)
#pragma unroll
                        for (int w = 0; w < WV; ++w) qy += popc64(Rx[w] & rows[y][w] & upper_mask(y, w));
                        M.pq[0][qn + popc64(bq & lanemask_lt())] = (rdense ? 1 << 25 : 0) | (qy << 16) | (xx << 8) | y;
                    }
                    qn += popc64(bq);
                }
                if (qn >= QRUN) drain();
            }
            if (qn > 0) drain();
            if (work) wk_ops += uni64(wave_sum(lops));
            const int64_t s24 = wave_sum(S);
            tacc.add((uint64_t)((int64_t)(wave_sum(lsum) + usum) + s24 / 24));
        };

        // W = 1: the same with one child per lane from many nodes of the task.
        // Lane x holds R = P & N+(x), taken apart by the lanes side by side (a
        // step takes the next y of every x) unless the wave counts it from its
        // missing pairs.  Queued children are the sets Q themselves.  (With a
        // queue per node, drained and summed up before the next one, an l = 4
        // node of Chung-Lu 3e5 took 870 vector instructions at k = 10, 17
        // children in 64 lanes: k = 8, 10, 11 19.9, 130, 143 ms against 14.7,
        // 101, 85 ms.)
        auto children1 = [&](const uint64_t (&P)[W], int l, int xhi) {
            if constexpr (W == 1) {
                const int lc = l - 2;
                q1_lc = lc;  // a task's leaves all have one parity
                if (l == 4 && xhi >= c) {
                    const int pc = popc64(P[0]);
                    bool pd = false;
                    if (pc < 4 || k4_missing(std::integral_constant<int, 1>{}, P, M.rows, pc, true, leaf_S, leaf_usum, pd))
                        return;
                }
                const int mycol = lane < c ? M.col[lane] : 0;
                const bool ax = ((P[0] >> lane) & 1) && lane < xhi && !(rule1 && mycol < l);
                uint64_t Rx = ax ? P[0] & dagv : 0;
                const int rx = popc64(Rx);
                if (rx < lc + 1) Rx = 0;
                if (work) {
                    const uint32_t rc = wsum_u32(Rx ? (uint32_t)rx : 0u);
                    wk_nodes += rc;
                    wk_ops += rc;
                }
                uint64_t dense = 0;  // lane x: bit 0 of its children's entries
                if (l == 5) {  // the larger sets by the wave
                    uint64_t big = uni64(ballot(Rx != 0 && rx >= L5_WAVE_MIN));
                    while (big) {
                        const int x = __builtin_ctzll(big);
                        big &= big - 1;
                        const uint32_t rlo = __builtin_amdgcn_readlane((uint32_t)Rx, x);
                        const uint32_t rhi = __builtin_amdgcn_readlane((uint32_t)(Rx >> 32), x);
                        const uint64_t R[1] = {((uint64_t)rhi << 32) | rlo};
                        bool rdense = false;
                        const bool done = k4_missing(std::integral_constant<int, 1>{}, R, M.rows, popc64(R[0]), false,
                                                     leaf_S, leaf_usum, rdense);
                        if (lane == x) {
                            dense = rdense ? 1 : 0;
                            if (done) Rx = 0;
                        }
                    }
                }
                uint64_t* q = M.q1[0];
                for (;;) {
                    const bool more = ballot(Rx != 0) != 0;
                    // (a shallow task has one such node: the queue ends with it)
                    if (q1 > Q1_RUN || (!DEEP && !more)) drain1();
                    if (!more) break;
                    bool ok = false;
                    uint64_t Q = 0;
                    if (Rx) {
                        const int y = __builtin_ctzll(Rx);
                        Rx &= Rx - 1;
                        Q = Rx & M.dag[y];
                        ok = popc64(Q) >= lc && !(rule1 && M.col[y] < l - 1);
                        if (popc64(Rx) < lc + 1) Rx = 0;
                    }
                    const uint64_t bq = ballot(ok);
                    if (ok) q[q1 + popc64(bq & lanemask_lt())] = Q | dense;
                    q1 += popc64(bq);
                }
            }
        };

        // Children of a node with l = 4 or 5 (x below xhi).  Classes
        // W = 2 and 3 first renumber a whole node whose candidate set fits
        // W - 1 words onto them (one narrower instance of the children and
        // leaf code per class keeps the kernel's spill space small), unless
        // the node is so small that renumbering (~6 W |P| instructions)
        // costs more than the narrower words save.
        auto count_children = [&](const uint64_t (&Pn)[W], int ln, int xhi) {
            if constexpr (W == 1) {
                children1(Pn, ln, xhi);
                return;
            }
            if constexpr (W == 2 || W == 3) {
                constexpr int WN = W - 1;
                const int p = popcW(Pn);
                if (xhi >= c && p <= 64 * WN && p >= COMPACT_MIN) {
                    uint64_t (*cr)[WN] = reinterpret_cast<uint64_t (*)[WN]>(M.crow);
                    compact_set<W, WN>(M, Pn, cr, M.ccol);
                    uint64_t Pc[WN];
                    prefix_mask<WN>(p, Pc);
                    children_by_lanes(std::integral_constant<int, WN>{}, Pc, cr, M.ccol, p, ln, 64 * WN);
                    return;
                }
            }
            if constexpr (W > 1) children_by_lanes(std::integral_constant<int, W>{}, Pn, M.rows, M.col, c, ln, xhi);
        };

        const int l0 = k - 2;
        uint64_t P0[W];
        prefix_mask<W>(c, P0);
        // A task covering the whole root may finish it in closed form; a
        // task holding only the root children with x below x1 counts
        // exactly the cliques of that part (so tasks can be listed alone).
        const bool whole = x1 >= c;
        bool active = true;
        int lq = 0;
        if (DEEP && qitem >= 0) {
            // a queued node (finish() already found no closed form for it)
            lq = uniform_i32(dev_load(&a.squeue[qitem].l));
        } else {
            // a root split over several tasks that is a clique, 2-plex or
            // 3-plex (as far as t allows): this task's part is the
            // l0-cliques whose first vertex x lies below x1, for a clique
            // sum_x C(c-1-x, l0-1), else the closed form of each later
            // neighbourhood P0 & N+(x) (a t-plex again) at l0 - 1
            const int xe = x1 < c ? x1 : c;
            bool close = whole;
            if (!whole && et && l0 >= 3) {
                int mn = 1 << 30;
#pragma unroll
                for (int q = 0; q < W; ++q) {
                    const int v = lane + 64 * q;
                    if (v < c) {
                        int d = 0;
#pragma unroll
                        for (int w = 0; w < W; ++w) d += popc64(P0[w] & M.rows[v][w]);
                        mn = d < mn ? d : mn;
                    }
                }
                const int mind = wmin_i32(mn);
                if (mind >= c - 1) {
                    val_t part = 0;
                    for (int x = 0; x < xe; ++x) part += choose(c - 1 - x, l0 - 1);
                    tacc.add(part);
                    active = false;
                } else {
                    close = mind >= c - tpl;
                }
            }
            if (close) {  // the whole root (x = -1), or its part vertex by vertex
                val_t part = 0;
                bool all = true;
                for (int x = whole ? -1 : 0; x < (whole ? 0 : xe) && all; ++x) {
                    uint64_t Rx[W];
#pragma unroll
                    for (int w = 0; w < W; ++w) Rx[w] = x < 0 ? P0[w] : uni64(P0[w] & M.rows[x][w] & upper_mask(x, w));
                    val_t v = 0;
                    all = finish(Rx, x < 0 ? l0 : l0 - 1, v);
                    part += v;
                }
                if (all) {
                    tacc.add(part);
                    active = false;
                }
            }
        }
        {
            const int lr = DEEP && qitem >= 0 ? lq : l0;
            if (active && (lr == 4 || lr == 5)) {
                uint64_t Pr[W];
#pragma unroll
                for (int w = 0; w < W; ++w) Pr[w] = DEEP && qitem >= 0 ? uni64(dev_load(&a.squeue[qitem].P[w])) : P0[w];
                count_children(Pr, lr, DEEP && qitem >= 0 ? c : x1);
                active = false;
            }
        }
        // hand node (Pn, ln), ln >= 4, to an idle wave through the queue
        // instead of searching it here; true when it was pushed
        // Whether waves wait for work is read from the counters (relaxed
        // loads, a round trip to L2) only every SQ_POLL_BUSY candidate nodes
        // while none wait and every SQ_POLL_HUNGRY while some do, and at
        // least every SQ_POLL_TICKS; in between the last answer stands.
        auto try_push = [&](const uint64_t (&Pn)[W], int ln) -> bool {
            if (!splitting || ln < 4) return false;
            const int pn = popcW(Pn);
            if (ln < 64 ? pn < __builtin_amdgcn_readlane(push_pmin, ln) : binom(pn, ln) < a.split_bound) return false;
            if (a.split_mode != SPLIT_FORCED) {
                if (poll_in > 0 && wall_clock64() - poll_t < SQ_POLL_TICKS) {
                    --poll_in;
                    if (!hungry) return false;
                } else {
                    poll_t = wall_clock64();
                    int hg = 0;
                    if (lane == 0) {
                        unsigned long long* sq = a.sq;
                        const unsigned long long r = dev_load(&sq[SQ_RESERVE]), h = dev_load(&sq[SQ_HEAD]);
                        hg = dev_load(&sq[SQ_IDLE]) > r - h;
                    }
                    hungry = uniform_i32(__shfl(hg, 0, 64)) != 0;
                    poll_in = hungry ? SQ_POLL_HUNGRY : SQ_POLL_BUSY;
                    if (!hungry) return false;
                }
            }
            int ok = 0;
            if (lane == 0) {
                unsigned long long* sq = a.sq;
                const unsigned long long r = dev_load(&sq[SQ_RESERVE]);
                if (r + SQ_SLACK < (unsigned long long)SQ_CAP) {
                    SplitItem& I = a.squeue[dev_add(&sq[SQ_RESERVE], 1ull)];
                    dev_store(&I.it, it);
#pragma unroll
                    for (int w = 0; w < W; ++w) dev_store(&I.P[w], Pn[w]);
                    dev_store(&I.l, (int32_t)ln);
                    wait_memory();
                    dev_store(&I.ready, 1);
                    sq_add(&sq[SQ_PUSHED], 1);
                    M.pushed = 1;
                    ok = 1;
                }
            }
            return uniform_i32(__shfl(ok, 0, 64)) != 0;
        };
        if constexpr (DEEP) {
        // depth-first search: the node being branched on lives in registers
        // (P, R, x, l); its ancestors are frames
        int sp = 0;
        uint64_t P[W], R[W];
        int x = -1, l = qitem >= 0 ? lq : l0;
#pragma unroll
        for (int w = 0; w < W; ++w) { P[w] = qitem >= 0 ? uni64(dev_load(&a.squeue[qitem].P[w])) : P0[w]; R[w] = 0; }
        while (active) {
            int y = -1;
            while (true) {
                bool any = false;
#pragma unroll
                for (int w = 0; w < W; ++w) any |= R[w] != 0;
                if (any) {
                    int wy = 0;
#pragma unroll
                    for (int w = W - 1; w >= 0; --w) if (R[w]) wy = w;
                    y = wy * 64 + __builtin_ctzll(R[wy]);
#pragma unroll
                    for (int w = 0; w < W; ++w) if (w == wy) R[w] &= R[w] - 1;
                    if (rule1 && M.col[y] < l - 1) {
#pragma unroll
                        for (int w = 0; w < W; ++w) R[w] = 0;
                        continue;
                    }
                    break;
                }
                int nx = -1;
#pragma unroll
                for (int w = W - 1; w >= 0; --w) {
                    const uint64_t b = P[w] & (x < 0 ? ~0ull : upper_mask(x, w));
                    if (b) nx = w * 64 + __builtin_ctzll(b);
                }
                const int xlim = sp == 0 ? x1 : c;
                if (nx < 0 || nx >= xlim || (rule1 && M.col[nx] < l)) { y = -1; break; }
                x = nx;
#pragma unroll
                for (int w = 0; w < W; ++w) R[w] = uni64(P[w] & M.rows[x][w] & upper_mask(x, w));
            }
            if (y < 0) {  // node exhausted: resume the parent
                if (sp == 0) break;
                --sp;
                Frame<W>& F = FR(sp);
#pragma unroll
                for (int w = 0; w < W; ++w) { P[w] = uni64(F.P[w]); R[w] = uni64(F.R[w]); }
                x = uniform_i32(F.x);
                l = uniform_i32(F.l);
                continue;
            }
            uint64_t Pc[W];
#pragma unroll
            for (int w = 0; w < W; ++w) Pc[w] = uni64(R[w] & M.rows[y][w] & upper_mask(y, w));
            const int lc = l - 2;
            if (work) wk_ops += W;
            if (popcW(Pc) < lc) continue;
            if (rule2 && lc >= 3) {
                if (work) wk_ops += W;
                int dc = 0;
#pragma unroll
                for (int q = 0; q < W; ++q) {
                    if (q >= ncq) break;
                    bool hit = false;
#pragma unroll
                    for (int w = 0; w < W; ++w) {
                        const int a0 = cs0[q] > 64 * w ? cs0[q] : 64 * w;
                        const int a1 = cs1[q] < 64 * w + 64 ? cs1[q] : 64 * w + 64;
                        if (a1 > a0) {
                            const int len = a1 - a0;
                            const uint64_t mk = (len == 64 ? ~0ull : ((1ull << len) - 1)) << (a0 - 64 * w);
                            hit |= (Pc[w] & mk) != 0;
                        }
                    }
                    dc += popc64(ballot(hit));
                }
                if (dc < lc) continue;
            }
            val_t v = 0;
            if (finish(Pc, lc, v)) { tacc.add(v); continue; }
            if (try_push(Pc, lc)) continue;
            if (lc == 4 || lc == 5) { count_children(Pc, lc, c); continue; }
            if (sp >= LDS_FRAMES + (gfr ? GLOBAL_FRAMES : 0)) {
                if (lane == 0) atomicOr(a.err, ERR_DEPTH);
                continue;
            }
            if (lane == 0 || sp >= LDS_FRAMES) {
                Frame<W>& F = FR(sp);
#pragma unroll
                for (int w = 0; w < W; ++w) { F.P[w] = P[w]; F.R[w] = R[w]; }
                F.x = x;
                F.l = l;
                F.y = y;
            }
            ++sp;
            wave_sync();
#pragma unroll
            for (int w = 0; w < W; ++w) { P[w] = Pc[w]; R[w] = 0; }
            x = -1;
            l = lc;
        }
        }

        if constexpr (W == 1) {
            if constexpr (DEEP) drain1();
            if (ballot(leaf_sum != 0 || leaf_S != 0) || leaf_usum) {
                const int64_t s24 = wave_sum(leaf_S);
                tacc.add((uint64_t)((int64_t)(wave_sum(leaf_sum) + leaf_usum) + s24 / 24));
            }
        }
        }
    task_done:
        // a batch flags an overflow on its own graph only (top bit of the
        // graph's high word), so co-scheduled graphs keep their results
        if (tacc.ovf && lane == 0) {
            if (a.graph_total) atomicOr(&a.graph_total[2 * gi + 1], 1ull << 63);
            else atomicOr(a.err, ERR_OVERFLOW);
        }
        if (a.per_task && lane == 0) a.per_task[it] = tacc.lo();  // (no splitting with per-task counts)
        if (a.graph_total) {
            if (lane == 0 && tacc.lo()) {
                const unsigned long long old = atomicAdd(&a.graph_total[2 * gi], (unsigned long long)tacc.lo());
                if (old + tacc.lo() < old) atomicAdd(&a.graph_total[2 * gi + 1], 1ull);
            }
            if (lane == 0 && tacc.hi()) atomicAdd(&a.graph_total[2 * gi + 1], (unsigned long long)tacc.hi());
        } else {
            acc.add(tacc.v);
        }
        wave_sync();
    }
    if (work && lane == 0) {
        atomicAdd(&a.work[0], (unsigned long long)wk_tasks);
        atomicAdd(&a.work[1], (unsigned long long)wk_nodes);
        atomicAdd(&a.work[2], (unsigned long long)wk_ops);
        if (a.wave_time) {
            const unsigned long long t1 = wall_clock64();
            atomicAdd(&a.wave_time[0], t1);
            atomicMax(&a.wave_time[1], t1);
            atomicAdd(&a.wave_time[2], 1ull);
            atomicMax(&a.wave_time[3], ~(unsigned long long)t_wave0);  // earliest start, complemented
        }
    }
    if (acc.ovf && lane == 0) atomicOr(a.err, ERR_OVERFLOW);
    if (lane == 0 && acc.v) {
        const unsigned long long old = atomicAdd(&a.total[0], (unsigned long long)acc.lo());
        const unsigned long long carry = (old + acc.lo() < old) ? 1ull : 0ull;
        if (acc.hi() + carry) atomicAdd(&a.total[1], (unsigned long long)(acc.hi() + carry));
    }
}

namespace {

// Workgroups per compute unit of the kernel, asked for once per device: the
// two calls took about 10 us of every launch.
template <int W, bool BUILD, bool DEEP>
int search_occupancy() {
    static std::atomic<int> known[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return -1;
    const bool slot = dev >= 0 && dev < 64;
    if (slot && known[dev].load(std::memory_order_acquire) > 0) return known[dev].load(std::memory_order_acquire);
    auto kern = k_search<W, BUILD, DEEP>;
    const size_t smem = 4 * sizeof(SearchMem<W>);
    if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem) != hipSuccess)
        return -1;
    int occ = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kern, 256, smem) != hipSuccess) return -1;
    if (occ < 1) occ = 1;
    if (slot) known[dev].store(occ, std::memory_order_release);
    return occ;
}

template <int W, bool BUILD, bool DEEP>
int64_t grid_blocks(int64_t ntasks, int cus, int blocks_per_cu) {
    int occ = search_occupancy<W, BUILD, DEEP>();
    if (occ < 0) return -1;
    if (blocks_per_cu > 0 && blocks_per_cu < occ) occ = blocks_per_cu;
    // blocks_per_cu = -2: one persistent workgroup per CU fewer than fit, so a
    // launch on another stream always finds room
    if (blocks_per_cu <= -2) occ = occ > 1 ? occ - 1 : 1;
    const int64_t need = (ntasks + 3) / 4;
    // blocks_per_cu = -1: one workgroup per four tasks, not persistent, so that
    // launches on other streams get compute units as workgroups retire
    int64_t grid = blocks_per_cu == -1 ? need : (int64_t)occ * cus;
    if (grid > need) grid = need;
    if (grid > 0x7fffffff) grid = 0x7fffffff;
    if (grid < 1) grid = 1;
    return grid;
}

template <int W, bool BUILD, bool DEEP>
hipError_t launch_w(SearchArgs a, int cus, int bpc, hipStream_t s) {
    const int64_t grid = grid_blocks<W, BUILD, DEEP>(a.ntasks, cus, bpc);
    if (grid < 0) return hipErrorInvalidValue;
    // tasks that build their sub-branch are sorted by graph, not by weight:
    // neighbours share the graph's arrays in cache
    a.tickets = make_tickets(a.next, a.ntasks, a.heavy, 4 * grid, BUILD ? 8 : 0, a.shared, bpc == -1);
    hipLaunchKernelGGL((k_search<W, BUILD, DEEP>), dim3((unsigned)grid), dim3(256), 4 * sizeof(SearchMem<W>), s, a);
    return hipGetLastError();
}

}  // namespace

template <int W>
hipError_t search_launch(bool build, const SearchArgs& a, int cus, int bpc, hipStream_t s) {
    if (a.deep) return build ? launch_w<W, true, true>(a, cus, bpc, s) : launch_w<W, false, true>(a, cus, bpc, s);
    return build ? launch_w<W, true, false>(a, cus, bpc, s) : launch_w<W, false, false>(a, cus, bpc, s);
}
// frames are sized for the deep searches, the only ones that have any
template <int W>
int64_t search_blocks(bool build, int64_t ntasks, int cus, int bpc) {
    return build ? grid_blocks<W, true, true>(ntasks, cus, bpc) : grid_blocks<W, false, true>(ntasks, cus, bpc);
}
template <int W>
hipError_t search_tables(hipStream_t s) {
    return launch_tables(s);
}

}  // namespace ebb
