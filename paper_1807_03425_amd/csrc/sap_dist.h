// Squared distances of a 64 x 64 tile of point pairs, in FP64 from direct
// differences (gfx950): the shared core of the one-time kernels that need
// 1/d^2 of every pair (the handle's tile array, the secant-PCA weights, the
// batched engine's tiles).
#pragma once

#include "sap_common.h"

namespace sap {

constexpr int kDistC = 16;           // components per staged chunk
constexpr int kDistS = kTile + 2;    // LDS row stride (doubles): 16-byte rows, writes two-way at most

// LDS of one tile: the row of X behind each of the tile's 64 + 64 points, and
// the staged chunk of both sides, component-major.
struct DistLds {
    int32_t row[2 * kTile];
    double x[2][kDistC][kDistS];
};

// Columns of a thread's block: two adjacent ones in each half of the tile, so
// that the 16 lanes of an LDS read of two columns cover every bank once (four
// adjacent ones would meet half of them twice).
__device__ __forceinline__ int tile_col(int tx, int c) { return 2 * tx + (c & 1) + 32 * (c >> 1); }

// d2[r][c] = sum_l (x_i - x_j)_l^2 for i = 4 ty + r of the tile's rows and
// j = tile_col(tx, c) of its columns, ty = tid / 16, tx = tid % 16 (256
// threads; all must call).  L.row holds the 128 rows of X (valid ones; the
// caller masks what lies past the end) and a barrier has made them visible.
//
// The differences are FP64 and the sum runs over l = 0, 1, .. in order, so a
// pair's value does not depend on its place in a tile.  Bound by FP64 VALU
// issue: 2 instructions per pair and component, against 4 LDS reads of 16
// bytes per 16 pairs.  At N = 20000, n = 200 3.3 ms (the issue floor is 2.0 ms
// at 2.4 GHz; under this load the card runs at 1.9, and 85% of the cycles
// issue); with a rounded square added at a time, 32 components per chunk and
// four adjacent columns per thread 4.7 ms; one pair per lane and 4 rows, the
// lane's column read from memory along n, 31.0 ms.  8 x 4 pairs per thread
// and half as many wavefronts: 3.4 ms, and slower by up to a third below 2000
// tiles.
template <typename TX>
__device__ __forceinline__ void tile_dist2(const TX *__restrict__ X, int64_t ldx, int n, DistLds &L,
                                           double (&d2)[4][4]) {
    const int c = threadIdx.x & (kDistC - 1), r0 = threadIdx.x / kDistC;   // staging: component, first row
    const int ty = threadIdx.x >> 4, tx = threadIdx.x & 15;
    constexpr int RS = 256 / kDistC, NR = kTile / RS;               // rows per step, steps
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int q = 0; q < 4; ++q) d2[r][q] = 0.0;
    // the chunk's loads, clamped to the row's last component (never used past it)
    TX v[2][NR];
    int row[2][NR];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int u = 0; u < NR; ++u) row[s][u] = L.row[s * kTile + r0 + u * RS];
    auto fetch = [&](int l0) __attribute__((always_inline)) {
        const TX *xl = X + min(l0 + c, n - 1);
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int u = 0; u < NR; ++u) v[s][u] = xl[row[s][u] * ldx];
    };
    fetch(0);
#pragma unroll 1
    for (int l0 = 0; l0 < n; l0 += kDistC) {
        if (l0 > 0) __syncthreads();   // the previous chunk has been read
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int u = 0; u < NR; ++u) L.x[s][c][r0 + u * RS] = (double)v[s][u];
        __syncthreads();
        if (l0 + kDistC < n) fetch(l0 + kDistC);
        const int nc = min(kDistC, n - l0);
#pragma unroll 4
        for (int l = 0; l < nc; ++l) {
            const double2 *pa = reinterpret_cast<const double2 *>(&L.x[0][l][4 * ty]);
            const double2 *pb = reinterpret_cast<const double2 *>(&L.x[1][l][2 * tx]);
            const double2 a0 = pa[0], a1 = pa[1], b0 = pb[0], b1 = pb[16];
            const double a[4] = {a0.x, a0.y, a1.x, a1.y}, b[4] = {b0.x, b0.y, b1.x, b1.y};
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const double t = a[r] - b[q];
                    d2[r][q] = __builtin_fma(t, t, d2[r][q]);
                }
        }
    }
}

// Whether the pair of rows xi, xj is shorter than min_len > 0, where d2 is
// tile_dist2's.  The length that decides is the root of the sum of rounded
// squares, as for the stored secants and the short pairs: it differs from d2
// by rounding only (2 (n + 1) 2^-53 of it at most), so it is formed where d2
// is that close to min_len^2, and where the square of min_len leaves the
// range.
template <typename TX>
__device__ __forceinline__ bool tile_shorter(const TX *__restrict__ xi, const TX *__restrict__ xj, int n, double d2,
                                             double min_len) {
    const double m2 = min_len * min_len;
    if (m2 > 1e-290 && fabs(d2 - m2) > (2.0 * n + 8.0) * 0x1p-52 * m2) return d2 < m2;
    double s = 0.0;
    for (int l = 0; l < n; ++l) {
        const double t = (double)xi[l] - (double)xj[l];
        s += t * t;
    }
    return sqrt(s) < min_len;
}

}  // namespace sap
