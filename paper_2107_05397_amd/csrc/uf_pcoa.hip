// Principal coordinates of a condensed distance matrix (gfx950).
//
// PCoA (Gower): A = -d^2/2, B = A - r 1^T - 1 r^T + g 11^T with r the row means
// of A (zero diagonal included) and g their mean; the coordinates are the top
// eigenvectors of B scaled by sqrt(eigenvalue).  B is never formed: every
// product B X is computed as
//     B X = A X - r (1^T X) - 1 (r^T X) + g 1 (1^T X),
// where A X reads the condensed matrix once per row block (HBM-bound).  The
// eigenpairs come from randomized subspace iteration with a Rayleigh-Ritz
// projection (Halko, Martinsson, Tropp 2011): Y = B Omega, then orthonormal
// bases of B Q, and T = Q^T B Q, whose small eigenproblem gives the Ritz pairs.
// Orthonormalisation is Cholesky QR, applied twice: from the Gram matrix G = Y^T Y =
// R^T R, Q = Y R^-1, leaving out columns that depend on others up to a relative floor
// (so rank-deficient B is handled).  All of it runs on the device; only the last
// eigenproblem, Q^T B Q, is solved on the host, by cyclic Jacobi rotations.  All
// reductions over samples run in a fixed order.  One call, 6,000 samples, 20 columns, 3
// iterations: 2.09 ms with SVQB (Stathopoulos and Wu 2002; the basis PCA still uses it)
// and its eigenproblems on the host, now 0.83; 300 samples 605 -> 237 us.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <numeric>
#include <type_traits>
#include <vector>

#include "uf.h"
#include "uf_internal.h"

namespace ufq {
namespace {

constexpr int kRB = 32;          // rows per block of the A X kernel
constexpr int kMaxCols = 48;     // columns of the test matrix (LDS: 33 KiB + up to 24 KiB)
constexpr int kSegs = 8;         // column-block segments of the A X kernel


typedef double v4d __attribute__((ext_vector_type(4)));

// Fixed-order block reduction of 256 doubles held one per thread.
__device__ __forceinline__ double block_sum(double v, double* red) {
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    const double s = red[0];
    __syncthreads();
    return s;
}

// sums[c] = sum_i X[i][c], sums[cols + c] = sum_i r_i X[i][c], by one block
__device__ __forceinline__ void col_sums(const double* __restrict__ X, int cols, int c, int64_t n,
                                         const double* __restrict__ rmean, double* __restrict__ sums,
                                         double* red) {
    double s = 0.0, t = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) {
        const double x = X[i * cols + c];
        s += x;
        t += rmean[i] * x;
    }
    s = block_sum(s, red);
    t = block_sum(t, red);
    if (threadIdx.x == 0) {
        sums[c] = s;
        sums[cols + c] = t;
    }
}

// P[seg][i][c] = sum over j in the segment, j != i, of (-d_ij^2 / 2) X[j][c], on
// v_mfma_f64_16x16x4_f64.  Block (ib, seg): 32 rows; its four waves take a quarter of
// the segment's steps of 16 columns j each and are added up in order at the end.  Lane l
// holds row l mod 16 of each 16-row group and columns 4 (l / 16) + t of the step (t = 0..3,
// one MFMA each), straight from the condensed matrix: above the diagonal its four
// values are consecutive, below it the 16 lanes' are.  Two to three waves
// a SIMD hide each other's loads.  NB: 16-column groups of X (zero past `cols`).  Blocks past the rows
// (grid.x > nblk) give the column sums of X (col_sums).
// Bound by reading the matrix, each element from both its row's and its column's block
// (6,000 samples: 288 MB, 3.8 TB/s; the MFMAs with 17-32 columns take 30 us of it).
// 6,000 samples, 20 columns: 138 us with the tile of A in LDS and FMAs from there, now
// 76; holding a step's values in registers over the next one's loads 84 (fewer waves).
constexpr int kAxWaves = 4;
constexpr int kAbove = 0, kBelow = 1, kAny = 2;
template <int NB>
__global__ __launch_bounds__(64 * kAxWaves, NB < 3 ? 2 : 1) void k_ax(const double* __restrict__ dm, int64_t n,
                                                      const double* __restrict__ X, int cols,
                                                      int64_t nblk, const double* __restrict__ rmean,
                                                      double* __restrict__ P, double* __restrict__ sums) {
    constexpr int RG = kRB / 16;
    __shared__ double red[kRB][NB * 16 + 1];
    if (int64_t(blockIdx.x) >= nblk) {
        const int c = int(blockIdx.x - nblk) * kSegs + int(blockIdx.y);
        if (c < cols) col_sums(X, cols, c, n, rmean, sums, &red[0][0]);
        return;
    }
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane & 15, grp = lane >> 4;
    const int64_t i0 = int64_t(blockIdx.x) * kRB;
    const int64_t nj = (n + 15) / 16, parts = int64_t(kSegs) * kAxWaves, part = int64_t(blockIdx.y) * kAxWaves + wave;
    const int64_t j_lo = nj * part / parts * 16, j_hi = nj * (part + 1) / parts * 16;
    v4d acc[RG][NB];
#pragma unroll
    for (int r = 0; r < RG; ++r)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[r][b] = v4d{0.0, 0.0, 0.0, 0.0};
    struct Step {
        double a[RG][4], x[NB][4];
    };
    // element (i, j) of the condensed matrix, i < j, is dm[at(i) + j]
    auto at = [&](int64_t i) { return i * n - i * (i + 1) / 2 - i - 1; };
    int64_t base[RG];
#pragma unroll
    for (int r = 0; r < RG; ++r) base[r] = at(min(i0 + 16 * r + row, n - 1));
    // mode: every column of the step above the diagonal of every row, below it, or any
    auto fetch = [&](auto mode_, int64_t j0) -> Step {
        constexpr int mode = decltype(mode_)::value;
        Step f;
#pragma unroll
        for (int r = 0; r < RG; ++r) {
            const int64_t i_first = i0 + 16 * r;
            if constexpr (mode == kAbove) {
                const double* from = dm + base[r] + j0 + 4 * grp;
#pragma unroll
                for (int t = 0; t < 4; ++t) f.a[r][t] = from[t];
            } else if constexpr (mode == kBelow) {
                const double* from = dm + at(j0 + 4 * grp) + min(i_first + row, n - 1);
                const int64_t step = n - 2 - (j0 + 4 * grp);     // at(j + 1) - at(j), one less each time
#pragma unroll
                for (int t = 0; t < 4; ++t) f.a[r][t] = from[t * step - t * (t - 1) / 2];
            } else {
                const int64_t i = i_first + row;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int64_t j = j0 + 4 * grp + t;
                    f.a[r][t] = i < n && j < n && i != j ? dm[i < j ? at(i) + j : at(j) + i] : 0.0;
                }
            }
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int64_t j = j0 + 4 * grp + t, jc = mode == kAny ? min(j, n - 1) : j;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const double x = X[jc * cols + min(16 * b + row, cols - 1)];
                f.x[b][t] = mode != kAny || j < n ? x : 0.0;
            }
        }
        return f;
    };
    bool col[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) col[b] = 16 * b + row < cols;
    auto use = [&](const Step& g) {   // (nothing reads a loaded value before this)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < RG; ++r) {
                const double a = 0.0 - 0.5 * g.a[r][t] * g.a[r][t];   // +0 where the distance is absent
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    acc[r][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, col[b] ? g.x[b][t] : 0.0, acc[r][b], 0, 0, 0);
            }
    };
    auto run = [&](auto mode_, int64_t lo, int64_t hi) {
        for (int64_t j0 = lo; j0 < hi; j0 += 16) use(fetch(mode_, j0));
    };
    const int64_t d_lo = min(max(i0, j_lo), j_hi);
    run(std::integral_constant<int, kBelow>{}, j_lo, d_lo);
    for (int64_t j0 = d_lo; j0 < min(i0 + kRB, j_hi); j0 += 16) use(fetch(std::integral_constant<int, kAny>{}, j0));
    const int64_t u_lo = max(j_lo, i0 + kRB), u_hi = min(j_hi, n / 16 * 16);
    run(std::integral_constant<int, kAbove>{}, u_lo, u_hi);
    for (int64_t j0 = max(u_lo, u_hi); j0 < j_hi; j0 += 16) use(fetch(std::integral_constant<int, kAny>{}, j0));
    for (int w = 0; w < kAxWaves; ++w) {
        if (wave == w) {
#pragma unroll
            for (int r = 0; r < RG; ++r)
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        double& to = red[16 * r + grp + 4 * q][16 * b + row];
                        to = w == 0 ? acc[r][b][q] : to + acc[r][b][q];
                    }
        }
        __syncthreads();
    }
    for (int e = threadIdx.x; e < kRB * cols; e += 64 * kAxWaves) {
        const int64_t i = i0 + e / cols;
        if (i < n) P[(int64_t(blockIdx.y) * n + i) * cols + e % cols] = red[e / cols][e % cols];
    }
}

hipError_t launch_ax(hipStream_t s, const double* dm, int64_t n, const double* X, int cols, int64_t nblk,
                     const double* rmean, double* P, double* sums) {
    const dim3 g{unsigned(nblk + (rmean ? (cols + kSegs - 1) / kSegs : 0)), unsigned(kSegs)};
    const dim3 t{64 * kAxWaves};
    if (cols <= 16) hipLaunchKernelGGL(k_ax<1>, g, t, 0, s, dm, n, X, cols, nblk, rmean, P, sums);
    else if (cols <= 32) hipLaunchKernelGGL(k_ax<2>, g, t, 0, s, dm, n, X, cols, nblk, rmean, P, sums);
    else if (cols <= kMaxCols) hipLaunchKernelGGL(k_ax<3>, g, t, 0, s, dm, n, X, cols, nblk, rmean, P, sums);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// r_i = (sum_seg P[seg][i]) / n (one column of ones)
__global__ __launch_bounds__(256) void k_row_means(const double* __restrict__ P, int64_t n,
                                                   double* __restrict__ r) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i >= n) return;
    double v = 0.0;
    for (int s = 0; s < kSegs; ++s) v += P[s * n + i];
    r[i] = v / double(n);
}

__global__ __launch_bounds__(256) void k_fill(double* __restrict__ p, int64_t n, double v) {
    const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (i < n) p[i] = v;
}

// Rows of a Gram block: 64-row tiles, at most kMaxGramBlocks blocks.
constexpr int kGT = 64;
constexpr int64_t kMaxGramBlocks = 128;
inline int64_t gram_rows(int64_t n) {
    const int64_t tiles = (n + kGT - 1) / kGT;
    return (tiles + kMaxGramBlocks - 1) / kMaxGramBlocks * kGT;
}
inline int64_t gram_blocks(int64_t n) { return (n + gram_rows(n) - 1) / gram_rows(n); }

// Gram entries of one tile in LDS (A^T B over its rows), added to the thread's; entry
// tid + 256 u of the c x c matrix
constexpr int kGE = (kMaxCols * kMaxCols + 255) / 256;
__device__ __forceinline__ void gram_tile(const double (*A)[kMaxCols + 1], const double (*B)[kMaxCols + 1],
                                          int c, double* g) {
#pragma unroll
    for (int u = 0; u < kGE; ++u) {
        const int e = threadIdx.x + 256 * u;
        if (e >= c * c) break;
        const int x = e / c, y = e % c;
        double v = g[u];
#pragma unroll 8
        for (int r = 0; r < kGT; ++r) v = fma(A[r][x], B[r][y], v);
        g[u] = v;
    }
}

// Y = sum_seg P[seg] - r (1^T X) - 1 (r^T X) + g 1 (1^T X), and the block's part of
// L^T Y (L null: Y^T Y) to Gp[block]
__global__ __launch_bounds__(256) void k_centre(const double* __restrict__ P, int64_t n, int c,
                                                const double* __restrict__ rmean,
                                                const double* __restrict__ gmean,
                                                const double* __restrict__ sums, int64_t rows,
                                                const double* __restrict__ L, double* __restrict__ Y,
                                                double* __restrict__ Gp) {
    __shared__ double ty[kGT][kMaxCols + 1], tl[kGT][kMaxCols + 1];
    const int64_t r0 = int64_t(blockIdx.x) * rows, r1 = min(n, r0 + rows);
    const double gm = gmean[0];
    double g[kGE];
#pragma unroll
    for (int u = 0; u < kGE; ++u) g[u] = 0.0;
    for (int64_t t0 = r0; t0 < r1; t0 += kGT) {
        __syncthreads();
        for (int e = threadIdx.x; e < kGT * c; e += 256) {
            const int r = e / c, k = e % c;
            const int64_t i = t0 + r;
            double y = 0.0, l = 0.0;
            if (i < r1) {
                double p[kSegs];
#pragma unroll
                for (int s = 0; s < kSegs; ++s) p[s] = P[(s * n + i) * c + k];
                double v = 0.0;
#pragma unroll
                for (int s = 0; s < kSegs; ++s) v += p[s];
                y = v - rmean[i] * sums[k] - sums[c + k] + gm * sums[k];
                if (L) l = L[i * c + k];
                Y[i * c + k] = y;
            }
            ty[r][k] = y;
            if (L) tl[r][k] = l;
        }
        __syncthreads();
        gram_tile(L ? tl : ty, ty, c, g);
    }
#pragma unroll
    for (int u = 0; u < kGE; ++u)
        if (threadIdx.x + 256 * u < c * c) Gp[int64_t(blockIdx.x) * c * c + threadIdx.x + 256 * u] = g[u];
}

// Q = Y M (M c x c), and the block's part of Q^T Q to Gp[block] (Gp null: none)
__global__ __launch_bounds__(256) void k_basis(const double* __restrict__ Y, int64_t n, int c,
                                               const double* __restrict__ M, int64_t rows,
                                               double* __restrict__ Q, double* __restrict__ Gp) {
    __shared__ double ty[kGT][kMaxCols + 1], tq[kGT][kMaxCols + 1], m[kMaxCols][kMaxCols + 1];
    const int64_t r0 = int64_t(blockIdx.x) * rows, r1 = min(n, r0 + rows);
    for (int e = threadIdx.x; e < c * c; e += 256) m[e / c][e % c] = M[e];
    double g[kGE];
#pragma unroll
    for (int u = 0; u < kGE; ++u) g[u] = 0.0;
    for (int64_t t0 = r0; t0 < r1; t0 += kGT) {
        __syncthreads();
        for (int e = threadIdx.x; e < kGT * c; e += 256)
            ty[e / c][e % c] = t0 + e / c < r1 ? Y[t0 * c + e] : 0.0;
        __syncthreads();
        for (int e = threadIdx.x; e < kGT * c; e += 256) {
            const int r = e / c, k = e % c;
            double v = 0.0;
            for (int t = 0; t < c; ++t) v = fma(ty[r][t], m[t][k], v);
            tq[r][k] = v;
            if (t0 + r < r1) Q[t0 * c + e] = v;
        }
        if (!Gp) continue;
        __syncthreads();
        gram_tile(tq, tq, c, g);
    }
    if (!Gp) return;
#pragma unroll
    for (int u = 0; u < kGE; ++u)
        if (threadIdx.x + 256 * u < c * c) Gp[int64_t(blockIdx.x) * c * c + threadIdx.x + 256 * u] = g[u];
}

// entry e of the sum of the c x c parts [b, e_b), in order
__device__ __forceinline__ double sum_parts(const double* __restrict__ Gp, int64_t b, int64_t b_end, int cc,
                                            int e) {
    double v = 0.0;
    for (; b < b_end; b += 16) {
        double p[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) p[u] = Gp[min<int64_t>(b + u, b_end - 1) * cc + e];
#pragma unroll
        for (int u = 0; u < 16; ++u) v += b + u < b_end ? p[u] : 0.0;
    }
    return v;
}
__global__ __launch_bounds__(256) void k_sum_parts(const double* __restrict__ Gp, int64_t nb, int cc,
                                                   double* __restrict__ T) {
    const int e = int(blockIdx.x) * 256 + threadIdx.x;
    if (e < cc) T[e] = sum_parts(Gp, 0, nb, cc, e);
}

// M (c x c, upper triangular) with (Y M)^T (Y M) = I but for the columns of Y that depend
// on earlier ones, which M makes zero (kept[j] = 0, else 1): from G = Y^T Y (nb parts) by
// Cholesky, G = R^T R, leaving out columns whose remaining norm is below a relative floor,
// and M = R^-1.  One block; one wave factorises, lane = column.  A chain of c steps, bound
// by their latency.  (The eigenvectors of G, found on the host, span the same space but
// cost two synchronisations and a Jacobi iteration each time: about 100 us with 20
// columns; this kernel 24.)
__global__ __launch_bounds__(1024) void k_chol(const double* __restrict__ Gp, int64_t nb, int c,
                                               double* __restrict__ M, double* __restrict__ kept) {
    __shared__ double G[kMaxCols][kMaxCols + 1], R[kMaxCols + 4][kMaxCols + 1], X[kMaxCols + 4][kMaxCols + 1];
    const int cc = c * c, half = cc <= 512 ? 512 : 0;   // two threads an entry where that fits
    for (int e = threadIdx.x; e < (kMaxCols + 4) * (kMaxCols + 1); e += 1024) (&R[0][0])[e] = (&X[0][0])[e] = 0.0;
    if (half) {
        const int e = threadIdx.x & 511;
        const bool second = threadIdx.x >= 512;
        const int64_t mid = (nb + 1) / 2;
        const double v = e < cc ? sum_parts(Gp, second ? mid : 0, second ? nb : mid, cc, e) : 0.0;
        if (!second && e < cc) G[e / c][e % c] = v;
        __syncthreads();
        if (second && e < cc) G[e / c][e % c] += v;
    } else {
        for (int e = threadIdx.x; e < cc; e += 1024) G[e / c][e % c] = sum_parts(Gp, 0, nb, cc, e);
    }
    __syncthreads();
    if (threadIdx.x < 64) {
        auto wave_sync = [] {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        };
        const int j = threadIdx.x, jc = min(j, kMaxCols - 1);
        double top = j < c ? G[j][j] : 0.0;
        const bool finite = __all(top < HUGE_VAL);      // else (also not a number) nothing is kept
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) top = fmax(top, __shfl_xor(top, o, 64));
        unsigned long long have = 0;
        for (int s = 0; s < c; ++s) {
            double v = j < c ? G[s][jc] : 0.0;
            for (int t = 0; t < s; t += 4)              // (rows past s are still zero)
#pragma unroll
                for (int u = 0; u < 4; ++u) v = fma(-R[t + u][s], R[t + u][jc], v);
            const double d = __shfl(v, s, 64);
            if (finite && d > 1e-14 * top) {
                have |= 1ull << s;
                if (j >= s && j < c) R[s][j] = v / sqrt(d);
            }
            wave_sync();
        }
        // column j of R^-1 from its end, over the columns kept
        for (int r = c - 1; r >= 0; --r) {
            if (!(have >> r & 1)) continue;
            double v = j == r ? 1.0 : 0.0;
            for (int t = r + 1; t < c; t += 4)          // (rows past c are zero)
#pragma unroll
                for (int u = 0; u < 4; ++u) v = fma(-R[r][min(t + u, kMaxCols)], X[t + u][jc], v);
            if (j < c && (have >> j & 1)) X[r][j] = v / R[r][r];
        }
        if (j < c) kept[j] = double(have >> j & 1);
    }
    __syncthreads();
    for (int e = threadIdx.x; e < cc; e += 1024) M[e] = X[e / c][e % c];
}

// G_part[b][x][y] = sum over rows of block b (kGramRows rows) of Y[i][x] Z[i][y]
constexpr int kGramRows = 128;

__global__ __launch_bounds__(256) void k_gram(const double* __restrict__ Y, int cy,
                                              const double* __restrict__ Z, int cz, int64_t n,
                                              double* __restrict__ Gp) {
    const int64_t b = blockIdx.x;
    const int64_t r0 = b * kGramRows, r1 = min(n, r0 + kGramRows);
    for (int e = threadIdx.x; e < cy * cz; e += 256) {
        const int x = e / cz, y = e % cz;
        double s = 0.0;
        for (int64_t i = r0; i < r1; ++i) s = fma(Y[i * cy + x], Z[i * cz + y], s);
        Gp[(b * cy + x) * cz + y] = s;
    }
}

// Q[i][:] = Y[i][:] M with M (cy x cq) row major, one thread per (i, column)
__global__ __launch_bounds__(256) void k_rightmul(const double* __restrict__ Y, int cy, int64_t n,
                                                  const double* __restrict__ M, int cq,
                                                  double* __restrict__ Q) {
    const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (e >= n * cq) return;
    const int64_t i = e / cq;
    const int c = int(e % cq);
    double s = 0.0;
    for (int k = 0; k < cy; ++k) s = fma(Y[i * cy + k], M[k * cq + c], s);
    Q[e] = s;
}

// Column k of V (n x dims): make its largest-magnitude entry (first on ties)
// positive.  One block per column; fixed-order arg-max.
__global__ __launch_bounds__(256) void k_signs(double* __restrict__ V, int dims, int64_t n) {
    __shared__ double bv[256];
    __shared__ int64_t bi[256];
    const int k = blockIdx.x;
    double best = -1.0;
    int64_t arg = 0;
    for (int64_t i = threadIdx.x; i < n; i += 256) {
        const double a = fabs(V[i * dims + k]);
        if (a > best) {
            best = a;
            arg = i;
        }
    }
    bv[threadIdx.x] = best;
    bi[threadIdx.x] = arg;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
            const double o = bv[threadIdx.x + w];
            const int64_t oi = bi[threadIdx.x + w];
            if (o > bv[threadIdx.x] || (o == bv[threadIdx.x] && oi < bi[threadIdx.x])) {
                bv[threadIdx.x] = o;
                bi[threadIdx.x] = oi;
            }
        }
        __syncthreads();
    }
    const bool flip = V[bi[0] * dims + k] < 0.0;
    if (!flip) return;
    for (int64_t i = threadIdx.x; i < n; i += 256) V[i * dims + k] = -V[i * dims + k];
}

// --------------------------------------------------------------------- host
// Eigen-decomposition of a symmetric m x m matrix by cyclic Jacobi rotations:
// on return a holds nothing useful, w the eigenvalues, v (row major, columns =
// eigenvectors).
void jacobi_eig(std::vector<double> a, int m, std::vector<double>& w, std::vector<double>& v) {
    v.assign(size_t(m) * m, 0.0);
    for (int i = 0; i < m; ++i) v[size_t(i) * m + i] = 1.0;
    auto A = [&](int i, int j) -> double& { return a[size_t(i) * m + j]; };
    double norm = 0.0;
    for (double x : a) norm += x * x;
    for (int sweep = 0; sweep < 100; ++sweep) {
        double off = 0.0;
        for (int i = 0; i < m; ++i)
            for (int j = i + 1; j < m; ++j) off += A(i, j) * A(i, j);
        if (off <= 1e-30 * norm || off == 0.0) break;
        for (int p = 0; p < m; ++p)
            for (int q = p + 1; q < m; ++q) {
                const double apq = A(p, q);
                if (apq == 0.0) continue;
                const double theta = (A(q, q) - A(p, p)) / (2.0 * apq);
                const double t = (theta >= 0 ? 1.0 : -1.0) /
                                 (std::fabs(theta) + std::sqrt(theta * theta + 1.0));
                const double c = 1.0 / std::sqrt(t * t + 1.0), s = t * c;
                for (int k = 0; k < m; ++k) {   // columns p, q
                    const double akp = A(k, p), akq = A(k, q);
                    A(k, p) = c * akp - s * akq;
                    A(k, q) = s * akp + c * akq;
                }
                for (int k = 0; k < m; ++k) {   // rows p, q
                    const double apk = A(p, k), aqk = A(q, k);
                    A(p, k) = c * apk - s * aqk;
                    A(q, k) = s * apk + c * aqk;
                }
                for (int k = 0; k < m; ++k) {
                    const double vkp = v[size_t(k) * m + p], vkq = v[size_t(k) * m + q];
                    v[size_t(k) * m + p] = c * vkp - s * vkq;
                    v[size_t(k) * m + q] = s * vkp + c * vkq;
                }
            }
    }
    w.resize(m);
    for (int i = 0; i < m; ++i) w[i] = A(i, i);
}

struct Plan {
    int64_t n = 0, nblk = 0;
    int cols = 0;
    size_t off_p = 0, off_y = 0, off_q = 0, off_z = 0, off_sums = 0, off_gp = 0, off_m = 0, off_t = 0,
           off_r = 0, off_g = 0, off_one = 0, total = 0;
};

size_t take(size_t& off, size_t bytes) {
    const size_t at = (off + 255) & ~size_t(255);
    off = at + bytes;
    return at;
}

Plan make_plan(int64_t n, int cols) {
    Plan p;
    p.n = n;
    p.cols = cols;
    p.nblk = (n + kRB - 1) / kRB;
    const size_t nc = size_t(n) * size_t(cols) * 8;
    size_t off = 0;
    p.off_p = take(off, nc * kSegs);
    p.off_y = take(off, nc);
    p.off_q = take(off, nc);
    p.off_z = take(off, nc);
    p.off_sums = take(off, size_t(2 * cols) * 8);
    p.off_gp = take(off, size_t(gram_blocks(n)) * cols * cols * 8);
    p.off_m = take(off, size_t(cols) * kMaxCols * 8);
    p.off_t = take(off, size_t(cols * cols + cols + 1) * 8);
    p.off_r = take(off, size_t(n) * 8);
    p.off_g = take(off, 8);
    p.off_one = take(off, size_t(n) * 8);
    p.total = off + 256;
    return p;
}

// ------------------------------------------------------------------ PCA basis
// Principal directions of a BF16 data matrix X [n][d] (row stride ldx): the
// same randomized subspace iteration, on the covariance C = Xc^T Xc / n with
// Xc = X - column means.  C is never formed: C Q = Xc^T (Xc Q).
constexpr int kPcaMaxCols = 160;   // columns of the test matrix
constexpr int kPcaT = 64;          // rows and columns of an X tile
constexpr int kPcaSplits = 8;      // row ranges of the X^T Y kernel

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float(uint32_t(h) << 16); }

// mu[j] = (1/n) sum_i X[i][j] (FP64, fixed order)
__global__ __launch_bounds__(256) void k_pca_mean(const uint16_t* __restrict__ X, int64_t ldx,
                                                  int64_t n, int64_t d, double* __restrict__ mu) {
    const int64_t j = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (j >= d) return;
    double s = 0.0;
    for (int64_t i = 0; i < n; ++i) s += double(bf16_to_f32(X[i * ldx + j]));
    mu[j] = s / double(n);
}

// Y[i][c] = sum_j (X[i][j] - mu[j]) Q[j][c] for a block of 64 rows.  Thread t
// owns row t/4 and columns t%4 + 4m; tiles of 64 columns of X (centred, FP32)
// and the matching 64 rows of Q (FP64) pass through LDS.
__global__ __launch_bounds__(256) void k_pca_xq(const uint16_t* __restrict__ X, int64_t ldx,
                                                int64_t n, int64_t d, const double* __restrict__ mu,
                                                const double* __restrict__ Q, int c,
                                                double* __restrict__ Y) {
    __shared__ float xs[kPcaT][kPcaT + 1];
    __shared__ double qs[kPcaT][kPcaMaxCols];
    const int t = threadIdx.x, r = t >> 2, g = t & 3;
    const int64_t i0 = int64_t(blockIdx.x) * kPcaT;
    constexpr int kM = kPcaMaxCols / 4;
    double acc[kM];
#pragma unroll
    for (int m = 0; m < kM; ++m) acc[m] = 0.0;
    for (int64_t j0 = 0; j0 < d; j0 += kPcaT) {
        for (int e = t; e < kPcaT * kPcaT; e += 256) {
            const int rr = e / kPcaT, jj = e % kPcaT;
            const int64_t i = i0 + rr, j = j0 + jj;
            xs[rr][jj] = (i < n && j < d) ? float(double(bf16_to_f32(X[i * ldx + j])) - mu[j]) : 0.0f;
        }
        for (int e = t; e < kPcaT * c; e += 256) {
            const int jj = e / c, cc = e % c;
            const int64_t j = j0 + jj;
            qs[jj][cc] = j < d ? Q[j * c + cc] : 0.0;
        }
        __syncthreads();
        for (int jj = 0; jj < kPcaT; ++jj) {
            const double xv = xs[r][jj];
#pragma unroll
            for (int m = 0; m < kM; ++m)
                if (g + 4 * m < c) acc[m] = fma(xv, qs[jj][g + 4 * m], acc[m]);
        }
        __syncthreads();
    }
    const int64_t i = i0 + r;
    if (i >= n) return;
#pragma unroll
    for (int m = 0; m < kM; ++m)
        if (g + 4 * m < c) Y[i * c + g + 4 * m] = acc[m];
}

// Zp[s][j][c] = sum over rows i of range s of (X[i][j] - mu[j]) Y[i][c], for a
// block of 64 columns j; thread t owns column t/4 and outputs t%4 + 4m.
__global__ __launch_bounds__(256) void k_pca_xty(const uint16_t* __restrict__ X, int64_t ldx,
                                                 int64_t n, int64_t d, const double* __restrict__ mu,
                                                 const double* __restrict__ Y, int c,
                                                 double* __restrict__ Zp) {
    __shared__ float xs[kPcaT][kPcaT + 1];     // [row i][column j]
    __shared__ double ys[kPcaT][kPcaMaxCols];
    const int t = threadIdx.x, jl = t >> 2, g = t & 3;
    const int64_t j0 = int64_t(blockIdx.x) * kPcaT;
    const int64_t per = (n + kPcaSplits - 1) / kPcaSplits;
    const int64_t ib = int64_t(blockIdx.y) * per, ie = min(n, ib + per);
    constexpr int kM = kPcaMaxCols / 4;
    double acc[kM];
#pragma unroll
    for (int m = 0; m < kM; ++m) acc[m] = 0.0;
    for (int64_t r0 = ib; r0 < ie; r0 += kPcaT) {
        for (int e = t; e < kPcaT * kPcaT; e += 256) {
            const int rr = e / kPcaT, jj = e % kPcaT;
            const int64_t i = r0 + rr, j = j0 + jj;
            xs[rr][jj] = (i < ie && j < d) ? float(double(bf16_to_f32(X[i * ldx + j])) - mu[j]) : 0.0f;
        }
        for (int e = t; e < kPcaT * c; e += 256) {
            const int rr = e / c, cc = e % c;
            const int64_t i = r0 + rr;
            ys[rr][cc] = i < ie ? Y[i * c + cc] : 0.0;
        }
        __syncthreads();
        for (int rr = 0; rr < kPcaT; ++rr) {
            const double xv = xs[rr][jl];
#pragma unroll
            for (int m = 0; m < kM; ++m)
                if (g + 4 * m < c) acc[m] = fma(xv, ys[rr][g + 4 * m], acc[m]);
        }
        __syncthreads();
    }
    const int64_t j = j0 + jl;
    if (j >= d) return;
    double* out = Zp + int64_t(blockIdx.y) * d * c;
#pragma unroll
    for (int m = 0; m < kM; ++m)
        if (g + 4 * m < c) out[j * c + g + 4 * m] = acc[m];
}

// Z = sum over the row ranges of Zp, in range order
__global__ __launch_bounds__(256) void k_pca_sum(const double* __restrict__ Zp, int64_t count,
                                                 double* __restrict__ Z) {
    const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (e >= count) return;
    double v = 0.0;
    for (int s = 0; s < kPcaSplits; ++s) v += Zp[s * count + e];
    Z[e] = v;
}

// out[r][j] = B[j][r] as FP32 (B: d x k FP64)
__global__ __launch_bounds__(256) void k_pca_out(const double* __restrict__ B, int64_t d, int k,
                                                 float* __restrict__ out) {
    const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (e >= d * k) return;
    const int64_t r = e / d, j = e % d;
    out[e] = float(B[j * k + r]);
}

struct PcaPlan {
    size_t off_mu = 0, off_y = 0, off_zp = 0, off_z = 0, off_q = 0, off_gp = 0, off_m = 0,
           off_b = 0, total = 0;
};

PcaPlan make_pca_plan(int64_t n, int64_t d, int c) {
    PcaPlan p;
    size_t off = 0;
    const int64_t rows = std::max(n, d);
    p.off_mu = take(off, size_t(d) * 8);
    p.off_y = take(off, size_t(n) * c * 8);
    p.off_zp = take(off, size_t(kPcaSplits) * d * c * 8);
    p.off_z = take(off, size_t(d) * c * 8);
    p.off_q = take(off, size_t(d) * c * 8);
    p.off_gp = take(off, size_t((rows + kGramRows - 1) / kGramRows) * c * c * 8);
    p.off_m = take(off, size_t(c) * c * 8);
    p.off_b = take(off, size_t(d) * c * 8);
    p.total = off + 256;
    return p;
}

}  // namespace
}  // namespace ufq

using ufh::fail;
using ufh::hip_fail;

#define UFQ_HIP(expr)                                     \
    do {                                                  \
        hipError_t e_ = (expr);                           \
        if (e_ != hipSuccess) return hip_fail(e_, #expr); \
    } while (0)

extern "C" {

uf_status uf_pcoa_workspace_size(int64_t n, int64_t n_cols, size_t* bytes) {
    if (!bytes) return fail(UF_ERR_ARG, "bytes is NULL");
    if (n < 2 || n_cols < 1 || n_cols > ufq::kMaxCols)
        return fail(UF_ERR_ARG, "need n >= 2 and 1 <= n_cols <= 48");
    *bytes = ufq::make_plan(n, int(std::min<int64_t>(n_cols, n))).total;
    return UF_OK;
}

uf_status uf_pcoa(const double* dm, int64_t n, const double* row_means, const double* grand_mean,
                  int64_t dims, int64_t n_cols, int power_iters, const double* omega,
                  double* coords, double* eigvals, double* trace, void* ws, size_t ws_bytes,
                  void* stream) {
    using namespace ufq;
    if (!dm || !omega || !coords || !eigvals) return fail(UF_ERR_ARG, "NULL argument");
    if (n < 2) return fail(UF_ERR_ARG, "need at least 2 samples");
    if (dims < 1 || n_cols < dims || n_cols > kMaxCols)
        return fail(UF_ERR_ARG, "need 1 <= dims <= n_cols <= 48");
    if (power_iters < 0 || power_iters > 64) return fail(UF_ERR_ARG, "power_iters in [0, 64]");
    if ((row_means == nullptr) != (grand_mean == nullptr))
        return fail(UF_ERR_ARG, "pass both row_means and grand_mean, or neither");
    int dev = 0;
    uf_status st = ufh::check_device(&dev);
    if (st != UF_OK) return st;
    const int l0 = int(n_cols);
    const int cols = int(std::min<int64_t>(n_cols, n));   // at most n independent directions
    const Plan p = make_plan(n, cols);
    if (!ws || ws_bytes < p.total) return fail(UF_ERR_WORKSPACE, "workspace missing or too small");
    hipStream_t s = static_cast<hipStream_t>(stream);
    char* base = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(ws) + 255) & ~uintptr_t(255));
    double* P = reinterpret_cast<double*>(base + p.off_p);
    double* Y = reinterpret_cast<double*>(base + p.off_y);
    double* Q = reinterpret_cast<double*>(base + p.off_q);
    double* Z = reinterpret_cast<double*>(base + p.off_z);
    double* sums = reinterpret_cast<double*>(base + p.off_sums);
    double* Gp = reinterpret_cast<double*>(base + p.off_gp);
    double* Md = reinterpret_cast<double*>(base + p.off_m);
    double* Td = reinterpret_cast<double*>(base + p.off_t);   // Q^T B Q, columns kept (1 or 0), mean of A
    const int64_t nbg = gram_blocks(n), rows = gram_rows(n);

    // row means of A and grand mean: given, or A 1 / n and its mean
    const double* rm = row_means;
    const double* gm = grand_mean;
    if (!rm) {
        double* r = reinterpret_cast<double*>(base + p.off_r);
        double* g = reinterpret_cast<double*>(base + p.off_g);
        double* one = reinterpret_cast<double*>(base + p.off_one);
        const dim3 gn{unsigned((n + 255) / 256)};
        hipLaunchKernelGGL(k_fill, gn, dim3(256), 0, s, one, n, 1.0);
        UFQ_HIP(hipGetLastError());
        UFQ_HIP(launch_ax(s, dm, n, one, 1, p.nblk, nullptr, P, sums));
        hipLaunchKernelGGL(k_row_means, gn, dim3(256), 0, s, P, n, r);
        UFQ_HIP(hipGetLastError());
        UFQ_HIP(ufk::grand_mean(r, n, g, s));
        rm = r;
        gm = g;
    }

    // B X (n x cols) into out, and the parts of L^T out (L null: out^T out)
    auto bx = [&](const double* X, const double* L, double* out) -> uf_status {
        UFQ_HIP(launch_ax(s, dm, n, X, cols, p.nblk, rm, P, sums));
        hipLaunchKernelGGL(k_centre, dim3(unsigned(nbg)), dim3(256), 0, s, P, n, cols, rm, gm, sums, rows, L,
                           out, Gp);
        UFQ_HIP(hipGetLastError());
        return UF_OK;
    };
    // out = the columns of Yin (whose Gram parts are in Gp) made orthonormal; again: leave
    // the Gram parts of out in Gp
    auto orth = [&](const double* Yin, double* out, bool again) -> uf_status {
        hipLaunchKernelGGL(k_chol, dim3(1), dim3(1024), 0, s, Gp, nbg, cols, Md, Td + cols * cols);
        UFQ_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_basis, dim3(unsigned(nbg)), dim3(256), 0, s, Yin, n, cols, Md, rows, out,
                           again ? Gp : nullptr);
        UFQ_HIP(hipGetLastError());
        return UF_OK;
    };

    // Omega is n x l0; a narrower basis (l0 > n) keeps its first `cols` columns
    const double* Om = omega;
    if (cols < l0) {
        std::vector<double> h(size_t(n) * l0), hs(size_t(n) * cols);
        UFQ_HIP(hipMemcpyAsync(h.data(), omega, h.size() * 8, hipMemcpyDeviceToHost, s));
        UFQ_HIP(hipStreamSynchronize(s));
        for (int64_t i = 0; i < n; ++i)
            for (int c = 0; c < cols; ++c) hs[size_t(i) * cols + c] = h[size_t(i) * l0 + c];
        UFQ_HIP(hipMemcpyAsync(Q, hs.data(), hs.size() * 8, hipMemcpyHostToDevice, s));
        UFQ_HIP(hipStreamSynchronize(s));   // hs goes out of scope
        Om = Q;
    }
    // Columns that a rank-deficient basis lacks are zero, and stay so.
    st = bx(Om, nullptr, Y);
    for (int it = 0; st == UF_OK; ++it) {
        st = orth(Y, Z, true);
        if (st == UF_OK) st = orth(Z, Q, false);
        if (st != UF_OK) return st;
        st = bx(Q, it < power_iters ? nullptr : Q, Y);
        if (it == power_iters) break;
    }
    if (st != UF_OK) return st;
    hipLaunchKernelGGL(k_sum_parts, dim3(unsigned((cols * cols + 255) / 256)), dim3(256), 0, s, Gp, nbg,
                       cols * cols, Td);
    UFQ_HIP(hipGetLastError());
    UFQ_HIP(hipMemcpyAsync(Td + cols * cols + cols, gm, 8, hipMemcpyDeviceToDevice, s));
    std::vector<double> ht(size_t(cols) * cols + cols + 1);
    UFQ_HIP(hipMemcpyAsync(ht.data(), Td, ht.size() * 8, hipMemcpyDeviceToHost, s));
    UFQ_HIP(hipStreamSynchronize(s));
    std::vector<int> have;   // columns of the basis
    for (int j = 0; j < cols; ++j)
        if (ht[size_t(cols) * cols + j] != 0.0) have.push_back(j);
    const int k = int(have.size());
    std::vector<double> lam(size_t(dims), 0.0);
    if (k > 0) {
        std::vector<double> W(size_t(cols) * dims, 0.0);   // cols x dims, scaled
        std::vector<double> T(size_t(k) * k), w, v;
        for (int a = 0; a < k; ++a)
            for (int b = 0; b < k; ++b)
                T[size_t(a) * k + b] = 0.5 * (ht[size_t(have[a]) * cols + have[b]] + ht[size_t(have[b]) * cols + have[a]]);
        jacobi_eig(T, k, w, v);
        std::vector<int> order(static_cast<size_t>(k));
        std::iota(order.begin(), order.end(), 0);
        std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return w[a] > w[b]; });
        for (int j = 0; j < dims && j < k; ++j) {
            const int o = order[size_t(j)];
            lam[size_t(j)] = w[size_t(o)];
            const double sc = std::sqrt(std::max(w[size_t(o)], 0.0));
            for (int r = 0; r < k; ++r) W[size_t(have[r]) * dims + j] = v[size_t(r) * k + o] * sc;
        }
        UFQ_HIP(hipMemcpyAsync(Md, W.data(), W.size() * 8, hipMemcpyHostToDevice, s));
        hipLaunchKernelGGL(k_rightmul, dim3(unsigned((n * dims + 255) / 256)), dim3(256), 0, s, Q, cols, n,
                           Md, int(dims), coords);
        UFQ_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_signs, dim3(unsigned(dims)), dim3(256), 0, s, coords, int(dims), n);
        UFQ_HIP(hipGetLastError());
        UFQ_HIP(hipStreamSynchronize(s));   // W goes out of scope
    } else {
        UFQ_HIP(hipMemsetAsync(coords, 0, size_t(n) * dims * 8, s));
        UFQ_HIP(hipStreamSynchronize(s));
    }
    std::memcpy(eigvals, lam.data(), size_t(dims) * 8);
    if (trace) *trace = -double(n) * ht[size_t(cols) * cols + cols];
    return UF_OK;
}


uf_status uf_pca_workspace_size(int64_t n, int64_t d, int64_t n_cols, size_t* bytes) {
    if (!bytes) return fail(UF_ERR_ARG, "bytes is NULL");
    if (n < 2 || d < 1 || n_cols < 1 || n_cols > ufq::kPcaMaxCols || n_cols > d)
        return fail(UF_ERR_ARG, "need n >= 2, d >= 1 and 1 <= n_cols <= min(160, d)");
    *bytes = ufq::make_pca_plan(n, d, int(n_cols)).total;
    return UF_OK;
}

uf_status uf_pca_basis(const void* x_bf16, int64_t n, int64_t d, int64_t ldx, int64_t k,
                       int64_t n_cols, int power_iters, const double* omega, float* basis,
                       double* eigvals, void* ws, size_t ws_bytes, void* stream) {
    using namespace ufq;
    if (!x_bf16 || !omega || !basis) return fail(UF_ERR_ARG, "NULL argument");
    if (n < 2 || d < 1 || ldx < d) return fail(UF_ERR_ARG, "need n >= 2, d >= 1 and ldx >= d");
    if (k < 1 || n_cols < k || n_cols > kPcaMaxCols || n_cols > d)
        return fail(UF_ERR_ARG, "need 1 <= k <= n_cols <= min(160, d)");
    if (power_iters < 0 || power_iters > 64) return fail(UF_ERR_ARG, "power_iters in [0, 64]");
    if (n > (int64_t(1) << 31) || d > (int64_t(1) << 24)) return fail(UF_ERR_ARG, "matrix too large");
    int dev = 0;
    uf_status st = ufh::check_device(&dev);
    if (st != UF_OK) return st;
    const int c = int(n_cols);
    const PcaPlan p = make_pca_plan(n, d, c);
    if (!ws || ws_bytes < p.total) return fail(UF_ERR_WORKSPACE, "workspace missing or too small");
    hipStream_t s = static_cast<hipStream_t>(stream);
    char* base = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(ws) + 255) & ~uintptr_t(255));
    const uint16_t* X = static_cast<const uint16_t*>(x_bf16);
    double* mu = reinterpret_cast<double*>(base + p.off_mu);
    double* Y = reinterpret_cast<double*>(base + p.off_y);
    double* Zp = reinterpret_cast<double*>(base + p.off_zp);
    double* Z = reinterpret_cast<double*>(base + p.off_z);
    double* Q = reinterpret_cast<double*>(base + p.off_q);
    double* Gp = reinterpret_cast<double*>(base + p.off_gp);
    double* Md = reinterpret_cast<double*>(base + p.off_m);
    double* B = reinterpret_cast<double*>(base + p.off_b);

    hipLaunchKernelGGL(k_pca_mean, dim3(unsigned((d + 255) / 256)), dim3(256), 0, s, X, ldx, n, d, mu);
    UFQ_HIP(hipGetLastError());
    // Y = Xc Qin (n x cq)
    auto xq = [&](const double* Qin, int cq) -> uf_status {
        hipLaunchKernelGGL(k_pca_xq, dim3(unsigned((n + kPcaT - 1) / kPcaT)), dim3(256), 0, s, X, ldx,
                           n, d, mu, Qin, cq, Y);
        UFQ_HIP(hipGetLastError());
        return UF_OK;
    };
    // Z = Xc^T Y (d x cq)
    auto xty = [&](int cq) -> uf_status {
        hipLaunchKernelGGL(k_pca_xty, dim3(unsigned((d + kPcaT - 1) / kPcaT), unsigned(kPcaSplits)),
                           dim3(256), 0, s, X, ldx, n, d, mu, Y, cq, Zp);
        UFQ_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_pca_sum, dim3(unsigned((d * cq + 255) / 256)), dim3(256), 0, s, Zp,
                           d * cq, Z);
        UFQ_HIP(hipGetLastError());
        return UF_OK;
    };
    // host copy of the fixed-order sum of A^T A over `rows` rows (ca x ca)
    auto gram = [&](const double* A, int ca, int64_t rows, std::vector<double>& G) -> uf_status {
        const int64_t nbg = (rows + kGramRows - 1) / kGramRows;
        hipLaunchKernelGGL(k_gram, dim3(unsigned(nbg)), dim3(256), 0, s, A, ca, A, ca, rows, Gp);
        UFQ_HIP(hipGetLastError());
        std::vector<double> part(size_t(nbg) * ca * ca);
        UFQ_HIP(hipMemcpyAsync(part.data(), Gp, part.size() * 8, hipMemcpyDeviceToHost, s));
        UFQ_HIP(hipStreamSynchronize(s));
        G.assign(size_t(ca) * ca, 0.0);
        for (int64_t b = 0; b < nbg; ++b)
            for (size_t e = 0; e < G.size(); ++e) G[e] += part[size_t(b) * G.size() + e];
        return UF_OK;
    };
    // SVQB of the d x cin matrix Ain into out (columns above the relative floor)
    auto svqb = [&](const double* Ain, int cin, double* out, int* kept) -> uf_status {
        std::vector<double> G, w, v;
        uf_status e = gram(Ain, cin, d, G);
        if (e != UF_OK) return e;
        jacobi_eig(G, cin, w, v);
        std::vector<int> order(static_cast<size_t>(cin));
        std::iota(order.begin(), order.end(), 0);
        std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return w[a] > w[b]; });
        const double top = cin > 0 ? w[size_t(order[0])] : 0.0;
        int kk = 0;
        while (kk < cin && top > 0.0 && w[size_t(order[size_t(kk)])] > 1e-14 * top) ++kk;
        *kept = kk;
        if (kk == 0) return UF_OK;
        std::vector<double> M(size_t(cin) * kk, 0.0);
        for (int j = 0; j < kk; ++j) {
            const int o = order[size_t(j)];
            const double sc = 1.0 / std::sqrt(w[size_t(o)]);
            for (int r = 0; r < cin; ++r) M[size_t(r) * kk + j] = v[size_t(r) * cin + o] * sc;
        }
        UFQ_HIP(hipMemcpyAsync(Md, M.data(), M.size() * 8, hipMemcpyHostToDevice, s));
        hipLaunchKernelGGL(k_rightmul, dim3(unsigned((d * kk + 255) / 256)), dim3(256), 0, s, Ain, cin,
                           d, Md, kk, out);
        UFQ_HIP(hipGetLastError());
        UFQ_HIP(hipStreamSynchronize(s));   // M is reused by the next call
        return UF_OK;
    };
    // Q <- orthonormal basis of Z's columns (SVQB twice, through B as scratch)
    auto orth = [&](int cin, int* kept) -> uf_status {
        int k1 = 0;
        uf_status e = svqb(Z, cin, B, &k1);
        if (e != UF_OK || k1 == 0) {
            *kept = k1;
            return e;
        }
        return svqb(B, k1, Q, kept);
    };

    int kq = 0;
    st = xq(omega, c);
    if (st != UF_OK) return st;
    st = xty(c);
    if (st != UF_OK) return st;
    st = orth(c, &kq);
    if (st != UF_OK) return st;
    for (int it = 0; it < power_iters && kq > 0; ++it) {
        st = xq(Q, kq);
        if (st != UF_OK) return st;
        st = xty(kq);
        if (st != UF_OK) return st;
        st = orth(kq, &kq);
        if (st != UF_OK) return st;
    }
    // Rayleigh-Ritz: H = (Xc Q)^T (Xc Q) = Q^T C Q n; its top eigenvectors W give
    // the directions Q W and the eigenvalues of C
    const int kk = int(std::min<int64_t>(k, kq));
    std::vector<double> lam(size_t(k), 0.0);
    std::vector<double> W(size_t(std::max(kq, 1)) * k, 0.0);
    if (kq > 0) {
        st = xq(Q, kq);
        if (st != UF_OK) return st;
        std::vector<double> H, w, v;
        const int64_t nbg = (n + kGramRows - 1) / kGramRows;
        hipLaunchKernelGGL(k_gram, dim3(unsigned(nbg)), dim3(256), 0, s, Y, kq, Y, kq, n, Gp);
        UFQ_HIP(hipGetLastError());
        {
            std::vector<double> part(size_t(nbg) * kq * kq);
            UFQ_HIP(hipMemcpyAsync(part.data(), Gp, part.size() * 8, hipMemcpyDeviceToHost, s));
            UFQ_HIP(hipStreamSynchronize(s));
            H.assign(size_t(kq) * kq, 0.0);
            for (int64_t b = 0; b < nbg; ++b)
                for (size_t e = 0; e < H.size(); ++e) H[e] += part[size_t(b) * H.size() + e];
        }
        jacobi_eig(H, kq, w, v);
        std::vector<int> order(static_cast<size_t>(kq));
        std::iota(order.begin(), order.end(), 0);
        std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return w[a] > w[b]; });
        for (int j = 0; j < kk; ++j) {
            const int o = order[size_t(j)];
            lam[size_t(j)] = w[size_t(o)] / double(n);
            for (int r = 0; r < kq; ++r) W[size_t(r) * k + j] = v[size_t(r) * kq + o];
        }
    }
    UFQ_HIP(hipMemcpyAsync(Md, W.data(), size_t(std::max(kq, 1)) * k * 8, hipMemcpyHostToDevice, s));
    if (kq > 0) {
        hipLaunchKernelGGL(k_rightmul, dim3(unsigned((d * k + 255) / 256)), dim3(256), 0, s, Q, kq, d,
                           Md, int(k), B);
        UFQ_HIP(hipGetLastError());
    } else {
        UFQ_HIP(ufk::zero_u32(reinterpret_cast<unsigned*>(B), 2 * d * k, s));
    }
    hipLaunchKernelGGL(k_pca_out, dim3(unsigned((d * k + 255) / 256)), dim3(256), 0, s, B, d, int(k),
                       basis);
    UFQ_HIP(hipGetLastError());
    UFQ_HIP(hipStreamSynchronize(s));   // W goes out of scope
    if (eigvals) std::memcpy(eigvals, lam.data(), size_t(k) * 8);
    return UF_OK;
}

}  // extern "C"
