// Squared distances of a 64 x 64 tile of point pairs, in FP64 from direct
// differences (gfx950): the shared core of the one-time kernels that need
// 1/d^2 of every pair (the handle's tile array, the secant-PCA weights, the
// batched engine's tiles).
#pragma once

#include "sap_common.h"

namespace sap {

constexpr int kDistC = 32;           // components per staged chunk
constexpr int kDistS = kTile + 2;    // LDS row stride (doubles): 16-byte rows, writes two-way at most

// LDS of one tile: the row of X behind each of the tile's 64 + 64 points, and
// the staged chunk of both sides, component-major.
struct DistLds {
    int32_t row[2 * kTile];
    double x[2][kDistC][kDistS];
};

// d2[r][c] = sum_l (x_i - x_j)_l^2 for i = 4 ty + r of the tile's rows and
// j = 4 tx + c of its columns, ty = tid / 16, tx = tid % 16 (256 threads; all
// must call).  L.row holds the 128 rows of X (valid ones; the caller masks
// what lies past the end) and a barrier has made them visible.
//
// The differences are FP64 and the sum runs over l = 0, 1, .. in order, a
// rounded square added at a time, so a pair's value does not depend on its
// place in a tile.  Bound by FP64 VALU issue: 3 instructions per pair and
// component (no FMA: its square would not be rounded), against 4 LDS reads of
// 16 bytes per 16 pairs.  The 4 x 4 block per thread is what makes it so: one
// pair per lane and 4 rows, with the lane's column read from memory along n
// (64 rows per load), took 31.0 ms at N = 20000, n = 200, where the issue
// floor is 3.1 ms; this form takes 4.7 ms.
template <typename TX>
__device__ __forceinline__ void tile_dist2(const TX *__restrict__ X, int64_t ldx, int n, DistLds &L,
                                           double (&d2)[4][4]) {
    const int c = threadIdx.x & (kDistC - 1), r0 = threadIdx.x / kDistC;   // staging: component, first row
    const int ty = threadIdx.x >> 4, tx = threadIdx.x & 15;
    constexpr int RS = 256 / kDistC, NR = kTile / RS;                      // rows per step, steps
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int q = 0; q < 4; ++q) d2[r][q] = 0.0;
    // the chunk's loads, clamped to the row's last component (never used past it)
    TX v[2][NR];
    auto fetch = [&](int l0) __attribute__((always_inline)) {
        const int lc = min(l0 + c, n - 1);
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int u = 0; u < NR; ++u) v[s][u] = X[(int64_t)L.row[s * kTile + r0 + u * RS] * ldx + lc];
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
            const double2 *pb = reinterpret_cast<const double2 *>(&L.x[1][l][4 * tx]);
            const double2 a0 = pa[0], a1 = pa[1], b0 = pb[0], b1 = pb[1];
            const double a[4] = {a0.x, a0.y, a1.x, a1.y}, b[4] = {b0.x, b0.y, b1.x, b1.y};
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const double t = a[r] - b[q];
                    d2[r][q] += t * t;
                }
        }
    }
}

}  // namespace sap
