// Internal declarations of the touched-branch pair tiles (uf_pairs.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstdint>

#include "uf_place.h"

namespace ufx {

constexpr int kPairA = 8;        // samples i per wave
constexpr int kPairWin = 256;    // branches listed at a time

// Workspace of one chunk of kc branches of n samples: values, then masks.
struct PairChunk {
    int64_t kcp = 0;             // masks per block
    size_t off_mask = 0, bytes = 0;
};
inline PairChunk pair_chunk(int64_t n, int64_t kc, size_t elem) {
    PairChunk c;
    const size_t nblk = size_t((n + 63) / 64);
    c.kcp = kc;
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
// m_ij of stripes [sb, se) over branches [ka, kb) of the chunk, `count` segments of
// seg branches side by side, each into its own plane of out: [se-sb][n] stripe-major,
// then sum_v x_iv of every sample i [n].  load: start from what out holds.
template <typename T>
hipError_t pairs(const void* chunk, int64_t n, int64_t kc, int64_t ka, int64_t kb, int64_t seg,
                 int64_t count, int64_t sb, int64_t se, int load, T* out, int64_t plane,
                 hipStream_t st);
// acc (first: =, else +=) the planes in order.
template <typename T>
hipError_t pair_planes(const T* planes, int64_t plane, int64_t count, int first, T* acc,
                       hipStream_t st);

}  // namespace ufx
