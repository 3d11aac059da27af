// Unweighted Gram product on presence bits and int8 matrix cores (gfx950):
//   G_ij = sum_v l_v a_iv a_jv  with l_v = q * (its fixed-point digits), a in {0, 1}.
//
// Presence is one bit per (sample, branch): samples in blocks of 64, one 64-bit word
// per (block, branch).  A branch's word is the OR of its tips' words, a contiguous
// range of tip ranks, taken from a 16-ary pyramid of ORs over the tips.
// Lengths are split into 7-bit digits d_0 .. d_{nd-1} (nd = 4 or 8), so that with
// operands in int8 and int32 sums the products a_i (a_j d) add exactly:
//   G_ij / q = sum_d 2^(7d) sum_v a_iv (a_jv d_v).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "uf_bits.h"
#include "uf_device.h"
#include "uf_internal.h"

namespace ufb {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef unsigned long long u64;

// one block per sample: its bit at the rank of each of its tips
__global__ __launch_bounds__(256) void k_tip_bits(int64_t pyr, const int64_t* __restrict__ row_ptr,
                                                  const int32_t* __restrict__ rank,
                                                  u64* __restrict__ tips) {
    const int64_t s = blockIdx.x;
    u64* t = tips + (s >> 6) * pyr;
    const u64 bit = 1ull << (s & 63);
    for (int64_t e = row_ptr[s] + threadIdx.x; e < row_ptr[s + 1]; e += 256) atomicOr(&t[rank[e]], bit);
}

// one pyramid level: each word ORs kFan words of the level below
__global__ __launch_bounds__(256) void k_or_level(int64_t pyr, int64_t from, int64_t n_from, int64_t to,
                                                  int64_t n_to, u64* __restrict__ tips) {
    const int64_t x = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (x >= n_to) return;
    u64* t = tips + int64_t(blockIdx.y) * pyr;
    u64 m = 0;
#pragma unroll
    for (int k = 0; k < kFan; ++k) {
        const int64_t y = x * kFan + k;
        m |= y < n_from ? t[from + y] : 0ull;
    }
    t[to + x] = m;
}

struct Levels {
    int64_t off[16];
};

// Word of every (block, branch of the chunk): the OR over tip ranks [lo, hi); and the
// branches of the block with a bit set, 64 to a word.
// The loose ends of a level, at most kFan - 1 on each side, then the level above; a
// random branch covers few tips, so most lanes end on the first level.
__global__ __launch_bounds__(256) void k_branch_bits(int64_t pyr, Levels lv, int64_t k0, int64_t kc,
                                                     const int32_t* __restrict__ lo,
                                                     const int32_t* __restrict__ hi,
                                                     const u64* __restrict__ tips, int64_t words,
                                                     u64* __restrict__ any, u64* __restrict__ bits) {
    const int64_t k = int64_t(blockIdx.x) * 256 + threadIdx.x;
    const u64* t = tips + int64_t(blockIdx.y) * pyr;
    int32_t l = k < kc ? lo[k0 + k] : 0, r = k < kc ? hi[k0 + k] : 0;
    u64 m = 0;
    for (int level = 0; l < r; ++level) {
        const u64* w = t + lv.off[level];
        if (r - l <= kFan) {
            for (; l < r; ++l) m |= w[l];
            break;
        }
        for (; l & (kFan - 1); ++l) m |= w[l];
        for (; r & (kFan - 1); --r) m |= w[r - 1];
        l /= kFan;
        r /= kFan;
    }
    if (k < kc) bits[int64_t(blockIdx.y) * kc + k] = m;
    const u64 touched = __ballot(m != 0ull);
    if ((threadIdx.x & 63) == 0 && (k >> 6) < words) any[int64_t(blockIdx.y) * words + (k >> 6)] = touched;
}

// 7-bit digits of rint(l / q), one per byte
__global__ __launch_bounds__(256) void k_digits(int kind, const double* __restrict__ len,
                                                const float* __restrict__ len32,
                                                const uint16_t* __restrict__ hi,
                                                const uint16_t* __restrict__ lo, double inv_q,
                                                int64_t k0, int64_t kc, u64* __restrict__ dig) {
    const int64_t k = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (k >= kc) return;
    const int64_t v = k0 + k;
    const double l = kind == 0   ? len[v]
                     : kind == 1 ? double(len32[v])
                                 : double(__uint_as_float(uint32_t(hi[v]) << 16)) +
                                       double(__uint_as_float(uint32_t(lo[v]) << 16));
    const u64 x = u64(llrint(l * inv_q));
    u64 d = 0;
#pragma unroll
    for (int b = 0; b < 8; ++b) d |= ((x >> (kDigitBits * b)) & 127ull) << (8 * b);
    dig[k] = d;
}

// bytes 0-3 (lo) or 4-7 (hi) of four words, transposed: out[c] holds byte c of each
__device__ __forceinline__ void transpose4(const uint32_t w[4], uint32_t out[4]) {
    const uint32_t a = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u);   // w0.0 w1.0 w0.1 w1.1
    const uint32_t b = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);   // w0.2 w1.2 w0.3 w1.3
    const uint32_t c = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u);
    const uint32_t d = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
    out[0] = __builtin_amdgcn_perm(c, a, 0x05040100u);
    out[1] = __builtin_amdgcn_perm(c, a, 0x07060302u);
    out[2] = __builtin_amdgcn_perm(d, b, 0x05040100u);
    out[3] = __builtin_amdgcn_perm(d, b, 0x07060302u);
}

// A workgroup owns a 64 x 64 tile of pairs: block bi of samples i, block bj of
// samples j.  Per window of kWin branches its threads list the branches that a sample
// of each block touches (32 branches per thread, from the words of touched branches).
// The list is staged kBatch branches at a time as LDS byte matrices [8][list] of the
// blocks' bits and [ND][list] of the length digits (four branches per thread,
// transposed in registers), so that 16 consecutive branches of 8 samples are one
// 16-byte read, and lane r turns them into int8 operands by a shift by r mod 8 and a
// mask.  The list's order does not matter: every sum is exact.
// Four waves: nd = 4: a 32 x 32 quarter of the tile each, all digits; nd = 8: a half
// of the i's and a half of the digits each, 64 j's.
//
// Why so.  The bits are 1/64 of FP64 values, so the operands of all tiles stay in L2;
// of the branches, 20 to 40% are touched on both sides of a 64 x 64 tile, and at int8
// rates a listed branch costs a tile 32 (nd 8) or 16 SIMD cycles, an eighth of what
// the vector units need.  It is bound by building operands beside the products: the matrix
// cores are busy in 48% of the SIMDs' busy cycles (nd 4, 5,000 samples x 100,000 tips; nd 8,
// 2,001 x 20,000: 47%).  Measured with events: FP64 2,001 samples x 20,000 tips 23.4 ms
// (vector kernel over all branches), 3.2 ms (pair tiles over touched branches) -> 0.32 ms;
// BF16 hi + lo lengths 5,000 x 100,000 7.4 ms (dense BF16 product over all branches) -> 2.2
// ms.  Listing with a ballot per 64 branches and byte stores per listed branch took 3.9 ms.
template <int ND>
__global__ __launch_bounds__(256, 2) void k_gram_bits(const u64* __restrict__ any,
                                                      const u64* __restrict__ bits,
                                                      const u64* __restrict__ dig, int64_t kc,
                                                      int64_t words, int64_t seg, ufd::TileSet tiles,
                                                      int64_t n, int64_t sb, int64_t se, int load,
                                                      double* __restrict__ out) {
    constexpr int NB = ND == 8 ? 2 : 1;     // 32-column blocks per wave
    constexpr int PITCH = kBatch + 32;      // rows 32 bytes apart modulo the banks
    __shared__ __attribute__((aligned(16))) uint8_t bi8[8][PITCH], bj8[8][PITCH], d8[ND][PITCH];
    __shared__ uint16_t list[kWin];
    __shared__ int wave_count[4];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int64_t bi, bj;
    if (!ufd::tile_of(tiles, blockIdx.x, bi, bj)) return;
    {
        // pairs of the tile in the stripe range: partner offset d = j - i; stripe d-1
        // if d <= S, else n-d-1
        const int64_t S = n / 2, i0 = bi * 64, j0 = bj * 64;
        const int64_t dlo = max<int64_t>(1, j0 - (min(i0 + 64, n) - 1)), dhi = min(j0 + 64, n) - 1 - i0;
        const int64_t a1 = max(dlo, sb + 1), b1 = min(dhi, min(se, S));
        const int64_t a2 = max(dlo, max(n - se, S + 1)), b2 = min(dhi, n - 1 - sb);
        // (a diagonal tile also gives its samples' own sums)
        if (bi != bj && (dhi < dlo || !(a1 <= b1 || a2 <= b2))) return;
    }
    const int ih = wave & 1, hh = wave >> 1;   // half of the i's; of the j's (nd 4) or digits (nd 8)
    const int jb0 = ND == 8 ? 0 : hh;
    const int dg0 = ND == 8 ? 4 * hh : 0;
    const int r = lane & 31, g = lane >> 5, sh = r & 7, row8 = r >> 3;
    v16i c[NB][4];
#pragma unroll
    for (int y = 0; y < NB; ++y)
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int e = 0; e < 16; ++e) c[y][d][e] = 0;

    const u64* wi = bits + bi * kc;
    const u64* wj = bits + bj * kc;
    const uint32_t* ai = reinterpret_cast<const uint32_t*>(any + bi * words);
    const uint32_t* aj = reinterpret_cast<const uint32_t*>(any + bj * words);
    const int64_t k_lo = seg * int64_t(blockIdx.y), k_hi = min(kc, k_lo + seg);
    for (int64_t w0 = k_lo; w0 < k_hi; w0 += kWin) {
        // this thread's 32 branches (words past the chunk hold no bits past its end)
        const int64_t kt = w0 + 32 * tid;
        uint32_t both = 0;
        if (kt < k_hi) both = ai[kt >> 5] & aj[kt >> 5];
        const int own = __popc(both);
        int inc = own;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(inc, off, 64);
            if (lane >= off) inc += o;
        }
        if (lane == 63) wave_count[wave] = inc;
        __syncthreads();                    // also: the previous list is consumed
        int at = inc - own, cnt = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const int o = wave_count[w];
            if (w < wave) at += o;
            cnt += o;
        }
        for (; both; both &= both - 1) list[at++] = uint16_t(32 * tid + __ffs(int(both)) - 1);
        __syncthreads();
        for (int b0 = 0; b0 < cnt; b0 += kBatch) {
            const int nb = min(kBatch, cnt - b0);
            if (4 * tid < nb + 32) {        // and up to 32 spare places
                u64 mi[4], mj[4], md[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int p = 4 * tid + u;
                    const int64_t k = w0 + list[b0 + min(p, nb - 1)];
                    mi[u] = wi[k];
                    mj[u] = wj[k];
                    md[u] = dig[k];
                    if (p >= nb) mi[u] = 0ull;   // no sample i: adds nothing
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    uint32_t w[4], o[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) w[u] = uint32_t(mi[u] >> (32 * h));
                    transpose4(w, o);
#pragma unroll
                    for (int q = 0; q < 4; ++q) *reinterpret_cast<uint32_t*>(&bi8[4 * h + q][4 * tid]) = o[q];
#pragma unroll
                    for (int u = 0; u < 4; ++u) w[u] = uint32_t(mj[u] >> (32 * h));
                    transpose4(w, o);
#pragma unroll
                    for (int q = 0; q < 4; ++q) *reinterpret_cast<uint32_t*>(&bj8[4 * h + q][4 * tid]) = o[q];
                    if (4 * h < ND) {
#pragma unroll
                        for (int u = 0; u < 4; ++u) w[u] = uint32_t(md[u] >> (32 * h));
                        transpose4(w, o);
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            *reinterpret_cast<uint32_t*>(&d8[(4 * h + q) % ND][4 * tid]) = o[q];
                    }
                }
            }
            __syncthreads();
            for (int t = 0; t < nb; t += 32) {
                const int x = t + 16 * g;
                const v4i pa = *reinterpret_cast<const v4i*>(&bi8[4 * ih + row8][x]);
                v4i a, m[NB];
#pragma unroll
                for (int e = 0; e < 4; ++e) a[e] = (pa[e] >> sh) & 0x01010101;
#pragma unroll
                for (int y = 0; y < NB; ++y) {
                    const v4i pb = *reinterpret_cast<const v4i*>(&bj8[4 * (jb0 + y) + row8][x]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const unsigned p = (unsigned(pb[e]) >> sh) & 0x01010101u;
                        m[y][e] = int((p << 8) - p);   // 0xFF where present
                    }
                }
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const v4i dv = *reinterpret_cast<const v4i*>(&d8[dg0 + d][x]);
#pragma unroll
                    for (int y = 0; y < NB; ++y)
                        c[y][d] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, m[y] & dv, c[y][d], 0, 0, 0);
                }
            }
            __syncthreads();                // the staged batch is consumed
        }
    }

    // D of a 32 x 32 block: lane holds column lane % 32, rows 8 (e / 4) + 4 (lane / 32) + e % 4
    const int64_t S = n / 2, sr = se - sb;
    out += int64_t(blockIdx.y) * (ND / 4) * (sr + 1) * n;
    if (ND == 8 && hh == 0) out += (sr + 1) * n;
#pragma unroll
    for (int y = 0; y < NB; ++y)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int64_t i = bi * 64 + 32 * ih + 8 * (e >> 2) + 4 * g + (e & 3);
            const int64_t j = bj * 64 + 32 * (jb0 + y) + r;
            if (!(i <= j && j < n)) continue;
            const int64_t d = j - i;
            const int64_t s = d == 0 ? se : d <= S ? d - 1 : n - d - 1;   // (w follows the stripes)
            if (d != 0 && (s < sb || s >= se)) continue;
            long long v = 0;
#pragma unroll
            for (int q = 3; q >= 0; --q) v = (v << kDigitBits) + (long long)c[y][q][e];
            const int64_t at = (s - sb) * n + (d <= S ? i : j);
            const double x = double(v) + (load ? out[at] : 0.0);
            out[at] = x;
            if ((n & 1) == 0 && d == S) out[(s - sb) * n + j] = x;   // the pair's other copy
        }
}

}  // namespace

hipError_t tip_bits(const ufp::Emb& e, int64_t n_tips, void* ws, hipStream_t st) {
    if (e.n <= 0) return hipSuccess;
    const BitsPlan p = bits_plan(e.n, n_tips, 0);
    if (p.nblk > 65535 || p.levels > 16) return hipErrorInvalidValue;
    u64* tips = static_cast<u64*>(ws);
    const int64_t n16 = (p.nblk * p.pyr * 8 + 15) / 16;   // (the bits of a chunk follow)
    hipError_t er = ufk::zero16(ws, n16, st);
    if (er != hipSuccess) return er;
    hipLaunchKernelGGL(k_tip_bits, dim3(unsigned(e.n)), dim3(256), 0, st, p.pyr, e.row_ptr, e.rank, tips);
    er = hipGetLastError();
    int64_t w = std::max<int64_t>(n_tips, 1);
    for (int64_t t = 1; t < p.levels && er == hipSuccess; ++t) {
        const int64_t to = (w + kFan - 1) / kFan;
        hipLaunchKernelGGL(k_or_level, dim3(unsigned((to + 255) / 256), unsigned(p.nblk)), dim3(256), 0,
                           st, p.pyr, p.level_off[t - 1], w, p.level_off[t], to, tips);
        er = hipGetLastError();
        w = to;
    }
    return er;
}

hipError_t branch_bits(const ufp::Emb& e, int64_t n_tips, int kind, const float* len32,
                       const uint16_t* len_hi, const uint16_t* len_lo, double inv_q, int64_t k0,
                       int64_t kc, void* ws, hipStream_t st) {
    if (e.n <= 0 || kc <= 0) return hipSuccess;
    const BitsPlan p = bits_plan(e.n, n_tips, kc);
    Levels lv;
    std::copy(p.level_off, p.level_off + 16, lv.off);
    char* base = static_cast<char*>(ws);
    hipLaunchKernelGGL(k_branch_bits, dim3(unsigned((kc + 255) / 256), unsigned(p.nblk)), dim3(256), 0, st,
                       p.pyr, lv, k0, kc, e.lo, e.hi, reinterpret_cast<const u64*>(base), p.words,
                       reinterpret_cast<u64*>(base + p.off_any), reinterpret_cast<u64*>(base + p.off_bits));
    hipError_t er = hipGetLastError();
    if (er != hipSuccess) return er;
    hipLaunchKernelGGL(k_digits, dim3(unsigned((kc + 255) / 256)), dim3(256), 0, st, kind, e.len, len32,
                       len_hi, len_lo, inv_q, k0, kc, reinterpret_cast<u64*>(base + p.off_dig));
    return hipGetLastError();
}

hipError_t gram_bits(int nd, int64_t n, int64_t n_tips, int64_t kc, int64_t splits, int64_t sb,
                     int64_t se, int load, double* out, const void* ws, hipStream_t st) {
    if (n <= 0 || kc <= 0 || se <= sb) return hipSuccess;
    const BitsPlan p = bits_plan(n, n_tips, kc);
    const ufd::TileSet tiles = ufd::tile_set(n, sb, se, true);
    const int64_t blocks = 8 * ((tiles.total + 7) / 8);
    const int64_t seg = ((kc + splits - 1) / splits + kSplit - 1) / kSplit * kSplit;
    // int32 sums: 127 per branch
    if (blocks > 0x7fffffff || splits < 1 || splits > 65535 || kc > (int64_t(1) << 23)) return hipErrorInvalidValue;
    const char* base = static_cast<const char*>(ws);
    const u64* any = reinterpret_cast<const u64*>(base + p.off_any);
    const u64* bits = reinterpret_cast<const u64*>(base + p.off_bits);
    const u64* dig = reinterpret_cast<const u64*>(base + p.off_dig);
    const dim3 grid{unsigned(blocks), unsigned(splits)};
    if (nd == 8)
        hipLaunchKernelGGL(k_gram_bits<8>, grid, dim3(256), 0, st, any, bits, dig, kc, p.words, seg, tiles, n, sb,
                           se, load, out);
    else if (nd == 4)
        hipLaunchKernelGGL(k_gram_bits<4>, grid, dim3(256), 0, st, any, bits, dig, kc, p.words, seg, tiles, n, sb,
                           se, load, out);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace ufb
