// Pair tiles over touched branches (gfx950), FP64 and FP32:
//   weighted    sum_v |x_iv - x_jv|    x = l u: branches that the tile's rows or columns touch
//   unweighted  sum_v min(x_iv, x_jv)  x = l a (the Gram value): branches that both touch
// so a tile of sample pairs leaves out the branches that add zero to all its pairs.
// (Weighted sums of minima, s_i + s_j - 2 m_ij, would need the shorter list too, but are a
// difference of large numbers: two samples of equal depth that differ on a few branches,
// d = 3e-9, are off by 2e-8 of their distance in FP64, and by all of it in FP32.)
//
// Chunk layout: samples in blocks of 64.  E[b][k][64] holds the block's values on
// branch k of the chunk (row kc is all zeros), mask[b][k] the bit of every sample
// of the block that touches it.
//
//   k_pair_fill    one walk over the branches every sample touches writes both
//   k_pairs        the tiles
//   k_pair_planes  adds the segments' sums in branch order
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "uf_device.h"
#include "uf_internal.h"
#include "uf_pairs.h"

namespace ufx {
namespace {

// One block per sample (tabs: of a batch of tables): every branch of [k0, k0 + kc) that the sample touches, once.
// Weighted: x = l c / T with the exact count c; unweighted: x = l.  Bound by the chain of
// the walks and by their scattered reads and writes.  With the row searched in memory and
// the node fields apart: 7,495 samples of eight tables, 20,000 branches 685 -> 547 us;
// 1,500 samples x 300 tips, 40,000 branches (FP64) 299 -> 204.
template <typename T, bool W>
__global__ __launch_bounds__(256) void k_pair_fill(ufp::Emb e, int32_t k0, int32_t kc,
                                                   const BatchTable* __restrict__ tabs,
                                                   const int32_t* __restrict__ tab_of,
                                                   T* __restrict__ E,
                                                   unsigned long long* __restrict__ mask) {
    // block b runs on XCD b mod 8: the samples of a 64-block on one XCD, whose L2 then
    // gathers the writes of their rows and masks
    const int64_t g = blockIdx.x >> 3, s = ((g >> 6) * 8 + (blockIdx.x & 7)) * 64 + (g & 63);
    if (s >= e.n) return;
    int64_t ls = s;      // in its table
    if (tabs) {
        const BatchTable t = tabs[tab_of[s]];
        ls = s - t.off;
        E += t.e_off;
        mask += t.m_off;
    }
    const int64_t a = e.row_ptr[s], b = e.row_ptr[s + 1];
    const double tot = e.total[s];
    T* Es = E + (ls >> 6) * (int64_t(kc) + 1) * 64 + (ls & 63);
    unsigned long long* ms = mask + (ls >> 6) * kc;
    const unsigned long long bit = 1ull << (ls & 63);
    if constexpr (W) {
        __shared__ ufd::RowLds row;
        ufd::for_each_counted_row_branch(e, e.nodes, row, s, [&](int32_t v, const int4&, auto&& count) {
            const int32_t k = v - k0;
            if (k < 0 || k >= kc) return;
            Es[int64_t(k) * 64] = T(e.len[v] * (double(count()) / tot));
            atomicOr(&ms[k], bit);
        });
    } else {
        for (int64_t ent = a + threadIdx.x; ent < b; ent += 256)
            ufd::for_each_branch(e, ent, a, [&](int32_t v) {
                const int32_t k = v - k0;
                if (k < 0 || k >= kc) return;
                Es[int64_t(k) * 64] = T(e.len[v]);
                atomicOr(&ms[k], bit);
            });
    }
}

// whether the pairs [i0, i1) x [j0, j1), i < j, hold one of stripes [sb, se)
__device__ __forceinline__ bool pairs_in_range(int64_t i0, int64_t i1, int64_t j0, int64_t j1,
                                               int64_t n, int64_t sb, int64_t se) {
    const int64_t S = n / 2;
    const int64_t dlo = max<int64_t>(1, j0 - (i1 - 1)), dhi = j1 - 1 - i0;
    if (dhi < dlo) return false;
    // partner offset d = j - i; stripe d-1 if d <= S, else n-d-1
    const int64_t a1 = max(dlo, sb + 1), b1 = min(dhi, min(se, S));
    const int64_t a2 = max(dlo, max(n - se, S + 1)), b2 = min(dhi, n - 1 - sb);
    return a1 <= b1 || a2 <= b2;
}

// value of lane L of the own 16-lane row
template <int L, typename T>
__device__ __forceinline__ T row_bcast(T v) {
    if constexpr (sizeof(T) == 8) {
        const long long b = __builtin_amdgcn_update_dpp(0ll, __double_as_longlong(v), 0x150 + L, 0xf, 0xf, true);
        return __longlong_as_double(b);
    } else {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + L, 0xf, 0xf, true));
    }
}

// min of two non-negative finite values, one instruction (FP32: their bits as
// integers, which order the same way)
__device__ __forceinline__ double vmin(double a, double b) {
    double d;
    asm("v_min_f64 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
    return d;
}
__device__ __forceinline__ float vmin(float a, float b) {
    return __uint_as_float(min(__float_as_uint(a), __float_as_uint(b)));
}

// descriptor over everything from p on (callers keep their offsets in range)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_of(const void* p) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, -4, 0x00027000);
}
template <typename T>
__device__ __forceinline__ T buf_load(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
    T o;
    if constexpr (sizeof(T) == 8) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, int(voff), int(soff), 0);
        __builtin_memcpy(&o, &v, 8);
    } else {
        const auto v = __builtin_amdgcn_raw_buffer_load_b32(r, int(voff), int(soff), 0);
        __builtin_memcpy(&o, &v, 4);
    }
    return o;
}

template <class F, int... I>
__device__ __forceinline__ void unrolled(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A wave owns A samples i x 64 samples j (one block).  Per window of kWin branches it
// lists those that one of its i and one of its j touch (from the masks, in branch
// order) in LDS, then runs the list in groups of U: lane l holds x_j of sample
// j0 + l, and the A values x_i, loaded into the lanes of every 16-lane row, are
// broadcast from there by DPP; an update is min and +.  Loads run one group ahead.
// A listed branch adds exactly its terms and the others add zero, so the sums
// are those over all branches in postorder, whichever tile a pair falls in.
// L1: sums of |x_i - x_j|, over the branches that either side touches; in FP32 two VALU
// operations an update with the broadcast in the first.
// blockIdx.y: segment [ka + seg*y, +seg) of the chunk, to its own plane of out.
//
// Why this shape.  A sample touches few branches (6% of a 20,000-tip tree at 300
// tips, 3% of a 200,000-tip tree at 1,000), but 64 samples together touch most, so
// a dense tile does mostly zeros: of the branches, 18% (8%) are touched on both sides
// of an 8 x 64 tile, and 56% (32%) on either side.  For minima, groups of 4 or 16
// samples i were slower (1,500 samples, 20,000 tips: 1.91 and 2.14 ms against 1.67), the
// first for its loads, the second for its longer lists.  Bound about half by FP64 issue
// (min, + or -, |+|, and one broadcast per A-row) and by L2 misses of the rows read.
// Measured with events as whole calls, against an LDS-tiled kernel over all branches
// (two workgroups of 128 x 128 pairs at 256 samples).  FP64 |x - y|: 256 samples, 1,000 tips
// 1.23 -> 0.083 ms; 1,500 x 20,000 24.9 -> 3.7; 5,000 x 5,000 17.5 -> 11.8; 8,000 x 5,000,
// most branches touched, 35.1 -> 31.6 (as sums of minima 0.076, 1.9, 8.9 and 40.1).  FP32:
// 500 x 2,000 branches 658 -> 43 us; 1,500 x 40,000 14.4 -> 2.15 ms; 5,000 x 10,000 8.8 ->
// 6.4 ms; 5,000 x 40,000 33.5 -> 16.5 ms, there bound by the rows that miss the caches;
// 10,000 x 2,000 5.4 -> 5.4.
constexpr int kWin = kPairWin;
// total (nullable): the sums go there instead, added to what it holds (more) or not.
template <typename T, int A, int U, bool L1>
__device__ __forceinline__ void pair_wave(uint32_t* q, const T* __restrict__ E,
                                          const unsigned long long* __restrict__ mask, int kc,
                                          int n, int64_t bi, int64_t bj, int ig, int k_lo,
                                          int k_hi, int sb, int se, bool load, T* out,
                                          T* total = nullptr, bool more = false) {
    constexpr int PER = 16 / A;             // branches per load of x_i
    constexpr int NI = U / PER;
    constexpr int ROW = 64 * int(sizeof(T));
    const int lane = threadIdx.x & 63;
    const int i0 = int(bi) * 64 + ig, j0 = int(bj) * 64;
    const int S = n / 2, j = j0 + lane;
    auto slot = [&](int a, int64_t* at, int64_t* dup) -> bool {
        const int i = i0 + a;
        *dup = -1;
        if (i >= j || j >= n) return false;
        const int d = j - i;
        const int s = d <= S ? d - 1 : n - d - 1;
        if (s < sb || s >= se) return false;
        const int64_t row = int64_t(s - sb) * n;
        *at = row + (d <= S ? i : j);
        if (!(n & 1) && d == S) *dup = row + j;   // an even N's last stripe holds the pair twice
        return true;
    };
    T r[A];
#pragma unroll
    for (int a = 0; a < A; ++a) {
        int64_t at, dup;
        r[a] = (load && slot(a, &at, &dup)) ? out[at] : T(0);
    }
    const T* Ei = E + bi * (int64_t(kc) + 1) * 64;
    const T* Ej = E + bj * (int64_t(kc) + 1) * 64;
    const uint32_t* mi = reinterpret_cast<const uint32_t*>(mask + bi * kc) + (ig >> 5);
    const unsigned long long* mj = mask + bj * kc;
    const unsigned ibits = ((1u << A) - 1u) << (ig & 31);
    const unsigned kl = unsigned(lane & 15) / A;
    const unsigned oi = unsigned(ig + (lane & (A - 1))) * unsigned(sizeof(T));
    const unsigned oj = unsigned(lane) * unsigned(sizeof(T));
    struct Group {
        T j[U], i[NI];
    };
    for (int w0 = k_lo; w0 < k_hi; w0 += kWin) {
        // the window's list; padded to whole groups with the zero row
        int cnt = 0;
        uint32_t a_[kWin / 64];
        unsigned long long b_[kWin / 64];
#pragma unroll
        for (int w = 0; w < kWin / 64; ++w) {
            const int k = min(w0 + 64 * w + lane, kc - 1);
            a_[w] = mi[2 * int64_t(k)];
            b_[w] = mj[k];
        }
#pragma unroll
        for (int w = 0; w < kWin / 64; ++w) {
            const int k = 64 * w + lane;
            const bool ti = (a_[w] & ibits) != 0u, tj = b_[w] != 0ull;
            const bool on = (L1 ? ti || tj : ti && tj) && w0 + k < k_hi;
            const unsigned long long bal = __ballot(on);
            const int at = cnt + int(__popcll(bal & ((1ull << lane) - 1ull)));
            if (on) q[at] = uint32_t(k);
            cnt += int(__popcll(bal));
        }
        if (lane < U) q[cnt + lane] = uint32_t(kc - w0);
        wave_sync();
        const __amdgpu_buffer_rsrc_t ri = buf_of(Ei + int64_t(w0) * 64);
        const __amdgpu_buffer_rsrc_t rj = buf_of(Ej + int64_t(w0) * 64);
        auto fetch = [&](int t) -> Group {
            Group g;
            const uint32_t ev = q[t * U + (lane & (U - 1))];
#pragma unroll
            for (int p = 0; p < NI; ++p)
                g.i[p] = buf_load<T>(ri, q[t * U + p * PER + kl] * unsigned(ROW) + oi, 0u);
#pragma unroll
            for (int u = 0; u < U; ++u)
                g.j[u] = buf_load<T>(rj, oj, unsigned(__builtin_amdgcn_readlane(int(ev), u)) * unsigned(ROW));
            return g;
        };
        auto use = [&](const Group& g) {
            unrolled([&](auto u_) {
                constexpr int u = decltype(u_)::value;
                unrolled([&](auto a_) {
                    constexpr int a = decltype(a_)::value;
                    const T xi = row_bcast<(u % PER) * A + a>(g.i[u / PER]);
                    if constexpr (L1) r[a] += fabs(xi - g.j[u]);
                    else r[a] += vmin(xi, g.j[u]);
                }, std::make_integer_sequence<int, A>{});
            }, std::make_integer_sequence<int, U>{});
        };
        const int ng = (cnt + U - 1) / U;
        if (ng > 0) {
            Group g0 = fetch(0), g1;
            for (int t = 0; t < ng; t += 2) {   // fetches past the last group re-read it
                g1 = fetch(min(t + 1, ng - 1));
                use(g0);
                g0 = fetch(min(t + 2, ng - 1));
                if (t + 1 < ng) use(g1);
            }
        }
        wave_sync();   // the list is rewritten next
    }
#pragma unroll
    for (int a = 0; a < A; ++a) {
        int64_t at, dup;
        if (!slot(a, &at, &dup)) continue;
        T* to = total ? total : out;
        const T v = more ? to[at] + r[a] : r[a];
        to[at] = v;
        if (dup >= 0) to[dup] = v;
    }
}

template <typename T, int A, bool L1>
__global__ __launch_bounds__(256) void k_pairs(const T* __restrict__ E,
                                               const unsigned long long* __restrict__ mask, int kc,
                                               ufd::TileSet tiles, int n, int sb, int se, int ka,
                                               int kb, int seg, int load, T* __restrict__ out,
                                               int64_t plane) {
    constexpr int SUB = 64 / (4 * A);
    constexpr int U = kPairU;
    __shared__ uint32_t queue[4][kWin + U];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int64_t bi, bj;
    const int64_t tb = blockIdx.x;
    if (!ufd::tile_of(tiles, ((tb >> 3) / SUB) * 8 + (tb & 7), bi, bj)) return;
    const int ig = (int((tb >> 3) % SUB) * 4 + wave) * A;     // first i inside its block
    const int i0 = int(bi) * 64 + ig, j0 = int(bj) * 64;
    if (i0 >= n) return;
    if (!pairs_in_range(i0, min(i0 + A, n), j0, min(j0 + 64, n), n, sb, se)) return;
    const int k_lo = ka + seg * int(blockIdx.y), k_hi = min(kb, k_lo + seg);
    pair_wave<T, A, U, L1>(queue[wave], E, mask, kc, n, bi, bj, ig, k_lo, k_hi, sb, se, load != 0,
                           out + int64_t(blockIdx.y) * plane);
}

// The same tiles over every table of a batch in one launch: items of 64 x 64 pairs and one
// segment, or (-1) all of the table's segments one after the other, 64 / A waves each; block
// b runs on XCD b mod 8 and so does its item.  A segment that an earlier chunk began goes on
// from its plane; last: the tree's branches end with this chunk.  ALL: items of all segments
// occur (compiled apart: the loop over them cost a batch without such items 4%).
// Every table's segments together fill the chip, so that its launches do not queue up
// behind small ones.  Eight tables of 300-1,500 samples x 20,000 branches, a whole call:
// 8.15 ms with 128 x 128 LDS tiles over all branches (about one workgroup of four waves
// per CU), now 3.9; three tables of 70-150 x 2,000: 0.78 -> 0.09 ms.  Waves that took
// their tiles from counters instead spent 0.37 ms per 4,096 waves on them.  The items of
// all tables in one list, cut in eighths by count: 7.5 ms (segments differ in length).
// Three tables of 4,500-9,000 samples x 40,000: 136 -> 84 ms, two of 9,000-16,000 x
// 100,000: 634 -> 340; 64 of 2,215-19,953 x 200,000: 33.6 -> 21.4 s.
template <int A, int U, bool ALL>
__global__ __launch_bounds__(256) void k_batch_pairs(const float* __restrict__ E,
                                                     const unsigned long long* __restrict__ mask,
                                                     const BatchTable* __restrict__ tabs,
                                                     const int4* __restrict__ items,
                                                     int k0, int kc, int last, float* __restrict__ acc) {
    constexpr int SUB = 64 / (4 * A);       // workgroups per item
    __shared__ uint32_t queue[4][kWin + U];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t tb = blockIdx.x;
    const int4 it = items[((tb >> 3) / SUB) * 8 + (tb & 7)];   // table, segment, block of i, block of j
    if (it.x < 0) return;
    const int ig = (int((tb >> 3) % SUB) * 4 + wave) * A;
    const BatchTable t = tabs[it.x];
    const int n = int(t.n);
    if (it.z * 64 + ig >= n) return;
    const bool all = ALL && it.y < 0;
    const int64_t g_end = all ? (int64_t(k0) + kc - 1) / t.seg : it.y;
    for (int64_t g = all ? k0 / t.seg : it.y; g <= g_end; ++g) {
        const int64_t s0 = g * t.seg;               // the segment's part in this chunk
        const int k_lo = int(max<int64_t>(s0 - k0, 0)), k_hi = int(min<int64_t>(s0 + t.seg - k0, kc));
        if (k_lo >= k_hi) return;
        const bool ends = all && (last || s0 + t.seg <= int64_t(k0) + kc);
        pair_wave<float, A, U, true>(queue[wave], E + t.e_off, mask + t.m_off, kc, n, it.z, it.w, ig, k_lo,
                                     k_hi, 0, n / 2, s0 < k0, acc + t.p_off + (all ? 0 : g) * t.plane,
                                     ends ? acc + t.acc_off : nullptr, ends && g > 0);
        if constexpr (!ALL) break;
    }
}

// Every table's sums: its segments' planes in order (tables of one segment have their
// sums there already).
__global__ __launch_bounds__(256) void k_batch_planes(const BatchTable* __restrict__ tabs,
                                                      float* __restrict__ acc) {
    const BatchTable t = tabs[blockIdx.y];
    if (t.n_seg < 2) return;
    for (int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x; e < t.plane; e += int64_t(gridDim.x) * 256) {
        float v = acc[t.p_off + e];
        for (int64_t p = 1; p < t.n_seg; ++p) v += acc[t.p_off + p * t.plane + e];
        acc[t.acc_off + e] = v;
    }
}

// acc (first: =, else +=) planes[0] + planes[1] + ..., in that order
template <typename T>
__global__ __launch_bounds__(256) void k_pair_planes(const T* __restrict__ planes, int64_t plane,
                                                     int count, int first, T* __restrict__ acc) {
    const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (e >= plane) return;
    T v = first ? planes[e] : acc[e] + planes[e];
    for (int p = 1; p < count; ++p) v += planes[p * plane + e];
    acc[e] = v;
}

// workgroups of k_pair_fill: whole groups of 8 x 64 samples
unsigned fill_blocks(int64_t n) { return unsigned((n + 511) / 512 * 512); }

}  // namespace

template <typename T>
hipError_t pair_fill(const ufp::Emb& e, int weighted, int64_t k0, int64_t kc, void* chunk,
                     hipStream_t st) {
    if (e.n <= 0 || kc <= 0) return hipSuccess;
    const PairChunk c = pair_chunk(e.n, kc, sizeof(T));
    T* E = static_cast<T*>(chunk);
    auto* mask = reinterpret_cast<unsigned long long*>(static_cast<char*>(chunk) + c.off_mask);
    const BatchTable* no_tabs = nullptr;
    const int32_t* no_tab_of = nullptr;
    const int64_t n16 = int64_t(c.bytes / 16);
    const hipError_t er = ufk::zero16(chunk, n16, st);
    if (er != hipSuccess) return er;
    if (weighted)
        hipLaunchKernelGGL((k_pair_fill<T, true>), dim3(fill_blocks(e.n)), dim3(256), 0, st, e,
                           int32_t(k0), int32_t(kc), no_tabs, no_tab_of, E, mask);
    else
        hipLaunchKernelGGL((k_pair_fill<T, false>), dim3(fill_blocks(e.n)), dim3(256), 0, st, e,
                           int32_t(k0), int32_t(kc), no_tabs, no_tab_of, E, mask);
    return hipGetLastError();
}

template <typename T, int A, bool L1>
static hipError_t pairs_as(const ufd::TileSet& tiles, const void* chunk, int64_t n, int64_t kc, int64_t ka, int64_t kb, int64_t seg,
                           int64_t count, int64_t sb, int64_t se, int load, T* out, int64_t plane,
                           hipStream_t st) {
    const PairChunk c = pair_chunk(n, kc, sizeof(T));
    const int64_t blocks = 8 * (64 / (4 * A)) * ((tiles.total + 7) / 8);
    if (blocks > 0x7fffffff || n > 0x7fffff00 || kc > 0x3fffffff || count > 65535)
        return hipErrorInvalidValue;
    const auto* mask = reinterpret_cast<const unsigned long long*>(static_cast<const char*>(chunk) + c.off_mask);
    hipLaunchKernelGGL((k_pairs<T, A, L1>), dim3(unsigned(blocks), unsigned(count)), dim3(256), 0, st,
                       static_cast<const T*>(chunk), mask, int(kc), tiles, int(n), int(sb), int(se),
                       int(ka), int(kb), int(std::min<int64_t>(seg, 0x3fffffff)), load, out, plane);
    return hipGetLastError();
}

template <typename T>
hipError_t pairs(int form, const void* chunk, int64_t n, int64_t kc, int64_t ka, int64_t kb, int64_t seg,
                 int64_t count, int64_t sb, int64_t se, int load, T* out, int64_t plane,
                 hipStream_t st) {
    if (n <= 0 || kb <= ka) return hipSuccess;
    const ufd::TileSet t = ufd::tile_set(n, sb, se, false);
    // (few stripes of a wide table: the narrower tiles, for twice the waves)
    const bool wide = n >= kPairWideN && t.total >= kPairWideN / 64 * (kPairWideN / 64) / 2;
    if (form == kPairL1)
        return wide ? pairs_as<T, 2 * kPairA, true>(t, chunk, n, kc, ka, kb, seg, count, sb, se, load, out, plane, st)
                    : pairs_as<T, kPairA, true>(t, chunk, n, kc, ka, kb, seg, count, sb, se, load, out, plane, st);
    if (form != kPairMin) return hipErrorInvalidValue;
    return pairs_as<T, kPairA, false>(t, chunk, n, kc, ka, kb, seg, count, sb, se, load, out, plane, st);
}

hipError_t batch_fill(const ufp::Emb& e, const BatchTable* tabs, const int32_t* tab_of, int64_t k0,
                      int64_t kc, void* chunk, size_t off_mask, size_t bytes, hipStream_t st) {
    if (e.n <= 0 || kc <= 0) return hipSuccess;
    if (kc > 0x3fffffff) return hipErrorInvalidValue;
    const int64_t n16 = int64_t((bytes + 15) / 16);
    const hipError_t er = ufk::zero16(chunk, n16, st);
    if (er != hipSuccess) return er;
    hipLaunchKernelGGL((k_pair_fill<float, true>), dim3(fill_blocks(e.n)), dim3(256), 0, st, e, int32_t(k0),
                       int32_t(kc), tabs, tab_of, static_cast<float*>(chunk),
                       reinterpret_cast<unsigned long long*>(static_cast<char*>(chunk) + off_mask));
    return hipGetLastError();
}

int batch_max_blocks(int stage_branches, int tile_stripes) {
    static const int limit[3][3] = {{5, 3, 2}, {3, 2, 2}, {1, 1, 1}};
    const int k = stage_branches == 8 ? 0 : stage_branches == 16 ? 1 : stage_branches == 32 ? 2 : -1;
    const int t = tile_stripes == 64 ? 0 : tile_stripes == 128 ? 1 : tile_stripes == 256 ? 2 : -1;
    return k < 0 || t < 0 ? 0 : limit[k][t];
}

template <int A, int U>
static hipError_t batch_pairs_as(const float* E, const unsigned long long* mask, const BatchTable* tabs,
                                 const int4* items, int64_t n_items, bool all, int64_t k0, int64_t kc,
                                 bool last, float* acc, hipStream_t st) {
    const int64_t blocks = (64 / (4 * A)) * n_items;
    if (blocks > 0x7fffffff || n_items % 8) return hipErrorInvalidValue;
    hipLaunchKernelGGL((all ? k_batch_pairs<A, U, true> : k_batch_pairs<A, U, false>), dim3(unsigned(blocks)),
                       dim3(256), 0, st, E, mask, tabs, items, int(k0), int(kc), int(last), acc);
    return hipGetLastError();
}

hipError_t batch_pairs(const void* chunk, size_t off_mask, const BatchTable* tabs, const int4* items,
                       int64_t n_items, bool all, int64_t k0, int64_t kc, bool last, float* acc,
                       int stage_branches, int tile_stripes, hipStream_t st) {
    const auto* E = static_cast<const float*>(chunk);
    const auto* mask = reinterpret_cast<const unsigned long long*>(static_cast<const char*>(chunk) + off_mask);
    if (n_items < 1 || kc < 1) return hipSuccess;
    if (kc > 0x3fffffff) return hipErrorInvalidValue;
#define UF_BP(KS_, TS_)                            \
    if (stage_branches == KS_ && tile_stripes == TS_) \
        return batch_pairs_as<TS_ / 16, KS_ / 2>(E, mask, tabs, items, n_items, all, k0, kc, last, acc, st);
    UF_BP(8, 64)
    UF_BP(8, 128)
    UF_BP(8, 256)
    UF_BP(16, 64)
    UF_BP(16, 128)
    UF_BP(16, 256)
    UF_BP(32, 64)
    UF_BP(32, 128)
    UF_BP(32, 256)
#undef UF_BP
    return hipErrorInvalidValue;
}

hipError_t batch_planes(const BatchTable* tabs, int64_t n_tables, int64_t max_plane, float* acc,
                        hipStream_t st) {
    if (n_tables < 1 || max_plane < 1) return hipSuccess;
    const unsigned gx = unsigned(std::min<int64_t>((max_plane + 255) / 256, 4096));
    for (int64_t r = 0; r < n_tables; r += 65535) {
        const unsigned gy = unsigned(std::min<int64_t>(n_tables - r, 65535));
        hipLaunchKernelGGL(k_batch_planes, dim3(gx, gy), dim3(256), 0, st, tabs + r, acc);
        const hipError_t er = hipGetLastError();
        if (er != hipSuccess) return er;
    }
    return hipSuccess;
}

template <typename T>
hipError_t pair_planes(const T* planes, int64_t plane, int64_t count, int first, T* acc,
                       hipStream_t st) {
    if (plane <= 0 || count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pair_planes<T>, dim3(unsigned((plane + 255) / 256)), dim3(256), 0, st, planes,
                       plane, int(count), first, acc);
    return hipGetLastError();
}

template hipError_t pair_fill<double>(const ufp::Emb&, int, int64_t, int64_t, void*, hipStream_t);
template hipError_t pair_fill<float>(const ufp::Emb&, int, int64_t, int64_t, void*, hipStream_t);
template hipError_t pairs<double>(int, const void*, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t,
                                  int64_t, int64_t, int, double*, int64_t, hipStream_t);
template hipError_t pairs<float>(int, const void*, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t,
                                 int64_t, int64_t, int, float*, int64_t, hipStream_t);
template hipError_t pair_planes<double>(const double*, int64_t, int64_t, int, double*, hipStream_t);
template hipError_t pair_planes<float>(const float*, int64_t, int64_t, int, float*, hipStream_t);

}  // namespace ufx
