// Device helpers shared by several kernel files: the embedded count of a
// sample on a branch, and the enumeration of the branches a sample touches.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "uf_place.h"

namespace ufd {

// first index in [a, b) whose tip rank is >= key
__device__ __forceinline__ int64_t lower_bound_rank(const int32_t* __restrict__ rank, int64_t a,
                                                    int64_t b, int32_t key) {
    while (a < b) {
        const int64_t mid = (a + b) >> 1;
        if (rank[mid] < key) a = mid + 1;
        else b = mid;
    }
    return a;
}

// sum of sample s's counts on the tips with rank in [lo, hi) (exact, integer)
__device__ __forceinline__ int64_t count_in(const ufp::Emb& e, int64_t s, int32_t lo, int32_t hi) {
    const int64_t a = e.row_ptr[s], b = e.row_ptr[s + 1];
    const int64_t p1 = lower_bound_rank(e.rank, a, b, lo);
    const int64_t p2 = lower_bound_rank(e.rank, p1, b, hi);
    return e.cum[p2 + s] - e.cum[p1 + s];
}

// The branches a sample touches, each exactly once: walking up from the tip
// of entry `entry`, branch v is reported when the previous tip of the row
// lies outside v's subtree (lo_v > rank[entry-1]); the walk stops at the first
// ancestor that also covers the previous tip.  The root is never reported.
template <typename F>
__device__ __forceinline__ void for_each_branch(const ufp::Emb& e, int64_t entry, int64_t row_start,
                                                F&& f) {
    const int32_t r = e.rank[entry];
    const int32_t prev = entry > row_start ? e.rank[entry - 1] : -1;
    int32_t v = e.tip_pos[r];
    int4 nd = e.nodes[v];
    while (v < e.root_pos && nd.x > prev) {
        const int4 up = e.nodes[nd.z];
        f(v);
        v = nd.z;
        nd = up;
    }
}

// A sample's row (tip ranks, exclusive prefix of the counts) in LDS.  Rows of up to
// kRowCap entries are staged there: the walks below search them at every branch, and
// from memory each probe of a search was a round trip of its own.
constexpr int kRowCap = 1024;
struct RowLds {
    int64_t cum[kRowCap + 1];
    int32_t rank[kRowCap];
};
__device__ __forceinline__ bool row_stage(const ufp::Emb& e, int64_t s, int64_t a, int64_t b, RowLds& L) {
    if (b - a > kRowCap) return false;
    const int m = int(b - a);
    for (int t = threadIdx.x; t <= m; t += blockDim.x) {
        L.cum[t] = e.cum[a + s + t];
        if (t < m) L.rank[t] = e.rank[a + t];
    }
    return true;
}

// The same branches with the sample's exact count on each where asked for: f(v, record,
// count()).  The sample's entries under a branch v of a walk are [entry, p2): none before
// lies under v (v does not cover the previous tip), and p2, the first entry at rank >=
// hi_v, only moves forward as the walk climbs, mostly by little, so it is searched for in
// steps of 1, 2, 4, ...  The parent's record is loaded while the branch is worked on.
// nodes: lo, hi, parent and a field of the caller's per position (one line a step).  LDS:
// the row is in L.
template <bool LDS, typename F>
__device__ __forceinline__ void for_each_counted_branch(const ufp::Emb& e, const int4* __restrict__ nodes,
                                                        const RowLds& L, int64_t s, int64_t a, int64_t b,
                                                        int entry, F&& f) {
    const int m = int(b - a);
    const int32_t* __restrict__ gr = e.rank + a;
    const int64_t* __restrict__ gc = e.cum + a + s;
    auto rank = [&](int t) -> int32_t {
        if constexpr (LDS) return L.rank[t];
        else return gr[t];
    };
    auto cum = [&](int t) -> int64_t {
        if constexpr (LDS) return L.cum[t];
        else return gc[t];
    };
    const int32_t prev = entry > 0 ? rank(entry - 1) : -1;
    int32_t v = e.tip_pos[rank(entry)];
    if (v >= e.root_pos) return;
    int4 nd = nodes[v];
    int p2 = entry + 1;
    while (nd.x > prev) {
        const int4 up = nodes[min(nd.z, e.root_pos - 1)];
        f(v, nd, [&]() -> int64_t {
            const int32_t hi = nd.y;
            if (p2 < m && rank(p2) < hi) {
                int from = p2 + 1, to = m;
                for (int w = 1;; w *= 2) {
                    const int t = from + w - 1;
                    if (t >= m) break;
                    if (rank(t) >= hi) {
                        to = t;
                        break;
                    }
                    from = t + 1;
                }
                while (from < to) {
                    const int mid = (from + to) >> 1;
                    if (rank(mid) < hi) from = mid + 1;
                    else to = mid;
                }
                p2 = from;
            }
            return cum(p2) - cum(entry);
        });
        v = nd.z;
        if (v >= e.root_pos) break;
        nd = up;
    }
}

// f over the walks of all entries of the row, by the block's threads.
template <typename F>
__device__ __forceinline__ void for_each_counted_row_branch(const ufp::Emb& e, const int4* __restrict__ nodes,
                                                            RowLds& L, int64_t s, F&& f) {
    const int64_t a = e.row_ptr[s], b = e.row_ptr[s + 1];
    const bool staged = row_stage(e, s, a, b, L);
    __syncthreads();
    const int m = int(b - a), step = int(blockDim.x);
    if (staged) {
        for (int t = threadIdx.x; t < m; t += step) for_each_counted_branch<true>(e, nodes, L, s, a, b, t, f);
    } else {
        for (int t = threadIdx.x; t < m; t += step) for_each_counted_branch<false>(e, nodes, L, s, a, b, t, f);
    }
}

// Tile t of the upper triangle of nblk x nblk blocks: super-tiles of G x G blocks,
// super-row-major, the diagonal super-tile first in its super-row, row-major inside.
// Workgroups are dealt to the 8 XCDs round-robin and XCD x takes the x-th eighth of
// that order, so its CUs walk neighbouring tiles (shared rows and columns in its L2).
constexpr int kTriGroup = 8;
__device__ __forceinline__ bool tri_tile(int64_t b, int64_t nblk, int64_t& bi, int64_t& bj) {
    constexpr int64_t G = kTriGroup;
    const int64_t L = nblk * (nblk + 1) / 2;
    const int64_t per = (L + 7) / 8;
    int64_t v = (b & 7) * per + (b >> 3);
    if ((b >> 3) >= per || v >= L) return false;
    for (int64_t r0 = 0;;) {
        const int64_t r = min(G, nblk - r0);
        const int64_t diag = r * (r + 1) / 2, cnt = diag + r * (nblk - r0 - r);
        if (v >= cnt) {
            v -= cnt;
            r0 += r;
            continue;
        }
        if (v < diag) {
            int64_t a = 0;
            while (v >= r - a) {
                v -= r - a;
                ++a;
            }
            bi = r0 + a;
            bj = bi + v;
        } else {
            v -= diag;
            const int64_t c0 = r0 + r + (v / (r * G)) * G;
            const int64_t c = min(G, nblk - c0);
            const int64_t w = v % (r * G);
            bi = r0 + w / c;
            bj = c0 + w % c;
        }
        return true;
    }
}

// The tiles of stripes [sb, se) of n samples: all of the triangle, or, where these are few,
// the diagonals bj - bi that the stripes' partner offsets [sb + 1, se] and [n - se, n - sb - 1]
// fall in (and, `self`, the tiles with bi = bj), 8 rows at a time.  Launching a workgroup for
// every tile of the triangle, most of them to end at once, took 0.3 ms at 20,000 samples.
struct TileSet {
    int64_t nblk = 0, total = 0;
    int64_t lo[3] = {0, 0, 0}, count[3] = {0, 0, 0};   // first diagonal and diagonals of each run
    bool all = true;
};
inline TileSet tile_set(int64_t n, int64_t sb, int64_t se, bool self) {
    TileSet t;
    t.nblk = (n + 63) / 64;
    t.total = t.nblk * (t.nblk + 1) / 2;
    // diagonal D holds offsets 64 D - 63 .. 64 D + 63
    int64_t from = 0, total = 0;
    auto run = [&](int k, int64_t first, int64_t last) {
        const int64_t a = first - 63 <= 0 ? 0 : first / 64;   // ceil((first - 63) / 64)
        t.lo[k] = a < from ? from : a;
        const int64_t hi = (last + 63) / 64 < t.nblk - 1 ? (last + 63) / 64 : t.nblk - 1;
        t.count[k] = hi >= t.lo[k] ? hi - t.lo[k] + 1 : 0;
        if (t.count[k] > 0) {
            from = hi + 1;
            total += t.count[k] * (t.nblk - t.lo[k]);
        }
    };
    if (self) run(0, 0, -63);
    run(1, sb + 1, se);
    run(2, n - se, n - sb - 1);
    if (2 * total <= t.total) {
        t.all = false;
        t.total = total;
    }
    return t;
}
// Tile b of 8 ceil(total / 8) workgroups (XCD b mod 8, as above); false: none.
__device__ __forceinline__ bool tile_of(const TileSet& t, int64_t b, int64_t& bi, int64_t& bj) {
    if (t.all) return tri_tile(b, t.nblk, bi, bj);
    const int64_t per = (t.total + 7) / 8;
    int64_t v = (b & 7) * per + (b >> 3);
    if ((b >> 3) >= per || v >= t.total) return false;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int64_t rows = t.nblk - t.lo[k], cnt = t.count[k] * rows;
        if (v < cnt) {
            const int64_t g = v / (kTriGroup * t.count[k]), r = v % (kTriGroup * t.count[k]);
            const int64_t h = min<int64_t>(kTriGroup, rows - g * kTriGroup);
            bi = g * kTriGroup + r % h;
            bj = bi + t.lo[k] + r / h;
            return bj < t.nblk;
        }
        v -= cnt;
    }
    return false;
}

}  // namespace ufd
