// Internal declarations of the touched-branch pair tiles (uf_pairs.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstdint>

#include "uf_internal.h"
#include "uf_place.h"

namespace ufx {

constexpr int kPairA = 8;        // samples i per wave
constexpr int kPairWin = 256;    // branches listed at a time
constexpr int kPairU = 8;        // branches per group of loads
constexpr int kPairMin = 0, kPairL1 = 1;   // sum of min(x, y); sum of |x - y|
// From here on the L1 tiles take 16 samples i per wave: their rows no longer stay in
// the caches, and each row of samples j read serves twice the pairs (FP32, 5,000 samples,
// 40,000 branches 28.2 -> 19.7 ms; 2,500: 6.5 -> 7.1; 1,500: 2.05 -> 2.37; FP64, 3,500:
// 17.8 -> 17.4, 2,500: 10.0 -> 11.2).  A batch runs such tables in a launch of their own.
constexpr int64_t kPairWideN = 4096;

// Workspace of one chunk of kc branches of n samples: values, then masks.
struct PairChunk {
    size_t off_mask = 0, bytes = 0;
};
inline PairChunk pair_chunk(int64_t n, int64_t kc, size_t elem) {
    PairChunk c;
    const size_t nblk = size_t((n + 63) / 64);
    c.off_mask = nblk * size_t(kc + 1) * 64 * elem;
    c.bytes = (c.off_mask + nblk * size_t(kc) * 8 + 15) / 16 * 16;
    return c;
}

// The branches' sum of a pair is taken in segments of this many branches (a fixed
// function of the table and tree sizes, so that every call on them adds in the same
// order): the whole tree at once when the tiles alone fill the chip, else up to 16
// segments that run side by side (6,144 waves fill 256 CUs six waves deep per SIMD;
// 256 samples on one segment of 2,000 branches take 113 us, on eight 29 us).
inline int64_t pair_segment(int64_t n, int64_t nb) {
    const int64_t nblk = (n + 63) / 64;
    const int64_t waves = nblk * (nblk + 1) / 2 * (64 / kPairA);
    const int64_t count = std::min<int64_t>(16, std::max<int64_t>(1, 6144 / std::max<int64_t>(waves, 1)));
    const int64_t len = (std::max<int64_t>(nb, 1) + count - 1) / count;
    return (len + kPairWin - 1) / kPairWin * kPairWin;
}

// Fill a chunk with branches [k0, k0 + kc) of every sample.
template <typename T>
hipError_t pair_fill(const ufp::Emb& e, int weighted, int64_t k0, int64_t kc, void* chunk,
                     hipStream_t st);
// Sums of stripes [sb, se) over branches [ka, kb) of the chunk, `count` segments of
// seg branches side by side, each into its own plane of out: [se-sb][n] stripe-major.
// load: start from what out holds.
template <typename T>
hipError_t pairs(int form, const void* chunk, int64_t n, int64_t kc, int64_t ka, int64_t kb, int64_t seg,
                 int64_t count, int64_t sb, int64_t se, int load, T* out, int64_t plane,
                 hipStream_t st);
// acc (first: =, else +=) the planes in order.
template <typename T>
hipError_t pair_planes(const T* planes, int64_t plane, int64_t count, int first, T* acc,
                       hipStream_t st);

// ---- batches: many tables on one tree, weighted, FP32 ----------------------
// Chunk of every table (PairChunk's layout per table: values at e_off, masks at
// off_mask + 8 m_off bytes), cleared (`bytes`) and filled.
hipError_t batch_fill(const ufp::Emb& e, const BatchTable* tabs, const int32_t* tab_of, int64_t k0,
                      int64_t kc, void* chunk, size_t off_mask, size_t bytes, hipStream_t st);
// The L1 tiles of every table on the chunk [k0, k0 + kc), segments each to its own
// plane at p_off.  items: (table, segment, block of 64 samples i, block of 64 samples
// j >= i), eight at a time, item p for XCD p mod 8 (table -1: none; segment -1, with `all`
// only: all, one after the other, their sums to acc_off as they end).  last: the chunk ends
// with the tree's branches.  Configuration: stage_branches (8, 16 or 32) branches in flight
// per wave; tiles of tile_stripes / 16 samples i (tile_stripes 64, 128 or 256) by 64 j.
hipError_t batch_pairs(const void* chunk, size_t off_mask, const BatchTable* tabs, const int4* items,
                       int64_t n_items, bool all, int64_t k0, int64_t kc, bool last, float* acc,
                       int stage_branches, int tile_stripes, hipStream_t st);
// The largest wgs_per_cu that a configuration may name (0: no such configuration): a
// fixed table, so that recorded configurations stay valid.  It sets nothing: as many waves
// run as fit (fewer, kept away by unused LDS, were slower by up to a fifth or the same).
int batch_max_blocks(int stage_branches, int tile_stripes);
// acc_off (=) the planes of each table, in order.
hipError_t batch_planes(const BatchTable* tabs, int64_t n_tables, int64_t max_plane, float* acc,
                        hipStream_t st);

}  // namespace ufx
