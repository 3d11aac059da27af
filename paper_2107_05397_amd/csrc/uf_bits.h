// Internal declarations of the unweighted Gram product on presence bits (uf_bits.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstdint>

#include "uf_place.h"

namespace ufb {

constexpr int kWin = 8192;         // branches listed at a time (32 per thread)
constexpr int kBatch = 1024;       // listed branches staged at a time (4 per thread)
constexpr int kDigitBits = 7;      // of a length digit (int8 operands, kept non-negative)
constexpr int kFan = 16;           // of the OR pyramid over the tips

// Workspace: bits of every tip and their OR pyramid; of one chunk of kc branches, the
// branches any sample of a block touches, the bits, and the length digits.
struct BitsPlan {
    int64_t nblk = 0, levels = 0, pyr = 0;   // blocks of 64 samples; pyramid levels and words per block
    int64_t level_off[16] = {};              // first word of each level
    int64_t words = 0;                       // 64-branch words of a chunk
    size_t off_any = 0, off_bits = 0, off_dig = 0, bytes = 0;
};
inline BitsPlan bits_plan(int64_t n, int64_t n_tips, int64_t kc) {
    BitsPlan p;
    p.nblk = (n + 63) / 64;
    for (int64_t w = std::max<int64_t>(n_tips, 1);; w = (w + kFan - 1) / kFan) {
        p.level_off[p.levels++] = p.pyr;
        p.pyr += w;
        if (w <= kFan) break;
    }
    p.words = (kc + 63) / 64;
    p.off_any = size_t(p.nblk * p.pyr) * 8;
    p.off_bits = p.off_any + size_t(p.nblk * p.words) * 8;
    p.off_dig = p.off_bits + size_t(p.nblk * kc) * 8;
    p.bytes = (p.off_dig + size_t(kc) * 8 + 15) / 16 * 16;
    return p;
}

constexpr int kSplit = 256;        // a range is a multiple of this

// Branch ranges that run side by side: enough blocks to fill the chip several times
// over (the sums are exact integers, so the split does not show in them).
inline int64_t bits_splits(int64_t n, int64_t kc) {
    const int64_t nblk = (n + 63) / 64, tiles = nblk * (nblk + 1) / 2;
    const int64_t most = (kc + kSplit - 1) / kSplit;
    return std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(16, most), 2048 / std::max<int64_t>(tiles, 1)));
}

// Bits of every tip and the pyramid (once per call).
hipError_t tip_bits(const ufp::Emb& e, int64_t n_tips, void* ws, hipStream_t st);
// Bits and digits of branches [k0, k0 + kc).  kind: the lengths (0: FP64, 1: FP32, 2:
// BF16 hi + lo), as rint(l / q) in nd digits.
hipError_t branch_bits(const ufp::Emb& e, int64_t n_tips, int kind, const float* len32,
                       const uint16_t* len_hi, const uint16_t* len_lo, double inv_q, int64_t k0,
                       int64_t kc, void* ws, hipStream_t st);
// G_ij / q of stripes [sb, se) and w_i / q = G_ii / q over the chunk's branches as exact
// integers in FP64 planes [se-sb+1][n], stripe-major, w last: nd = 4: one plane (digits
// 0-3); nd = 8: the plane of digits 4-7 (in units of 2^28), then that of digits 0-3.  Split
// y writes its own planes at out + y * (planes of one split); load: add to what out holds.
hipError_t gram_bits(int nd, int64_t n, int64_t n_tips, int64_t kc, int64_t splits, int64_t sb,
                     int64_t se, int load, double* out, const void* ws, hipStream_t st);

}  // namespace ufb
