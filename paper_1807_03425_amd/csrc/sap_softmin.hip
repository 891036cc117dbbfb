// Soft-min surrogate of the minimum projected unit-secant norm, and its
// gradient in P (gfx950).  Not part of the paper's method: a differentiable
// stand-in for its min, for gradient-based optimisation of P.
//
//   L      = -tau log sum_{kept i<j} exp(-r_ij / tau),   r_ij = ||P^T s_ij||
//   dL/dP  = sum w_ij s_ij (P^T s_ij)^T / r_ij,          w_ij = exp(-(r_ij - L)/tau)
//
// With Y = (X - mu) P, y_i - y_j = P^T (x_i - x_j), and d_ij = ||x_i - x_j||,
// s (P^T s)^T / r = (x_i - x_j)(y_i - y_j)^T / (d^2 r), so the gradient is a
// weighted graph Laplacian contraction:
//   dL/dP = (X - mu)^T Z,   z_i = sum_{j != i} a_ij (y_i - y_j),
//   a_ij  = w_ij (1/d_ij^2) / r_ij   (0 when r_ij = 0).
// The weights a_ij are recomputed tile by tile from Y and the stored 1/d^2
// (never stored), in the same 64 x 64 tile order as the pair pass.  Pairs on
// the short-pair list (fused form) are evaluated from their FP64 difference
// vectors, as in the iteration.
//
// Launch sequence
//   forward:  k_sm_loadP   P (FP32, n x k) -> FP64 k x n, and a copy
//             k_sm_prep    Y = (X - mu) P (FP64 MFMA, rounded to FP32) and the
//                          FP64 (min, sum) partials of the short pairs
//             k_sm_fwd     per-block (min, scaled sum) over the tiles
//             k_sm_fin     one block: merge in FP64, L, loss
//   backward: k_sm_same    P against the forward's
//             k_sm_prep    (short-pair blocks only) a_ij (y_i - y_j) per short pair
//             k_sm_bwd     partial z sums of rows (per share: half-tiles of a
//                          row of tiles) and columns (per tile) -- weights and
//                          column side on VALU, row-side contraction on FP64 MFMA
//             k_sm_zred    z_i per point: partials + short pairs, FP64
//             k_sm_grad    (X - mu)^T Z per row chunk, FP64 MFMA
//             k_sm_dP      sum of the chunks times dL/dloss
#include "sap_common.h"

namespace sap {

// log-sum-exp state: reference m and s = sum exp(-(r - m)/tau); s == 0 means
// empty (m is then ignored)
struct SmPart {
    double m, s;
};

struct SmArgs {
    const float *Y;        // soft-min Y, Npad x kp
    int kp;
    const float4 *invd2;
    const int2 *tiles;
    int64_t nhalf;
    int npass;             // pass blocks; their partials come first in `part`
    int n;
    // short pairs
    const int2 *close;
    const double *cd;
    int64_t nclose;
    // parameters
    const double *P64t;    // soft-min P, k x n FP64
    int vx, vp;            // 16-byte loads: X rows aligned; n even
    int gemm;              // arithmetic of the Y GEMM (SAP_GEMM_*)
    double tau;
    float c2;              // log2(e) / tau
    double c2d;            // the same in FP64
    SmPart *part;          // npass + nshort partials (forward)
    const double *Lp, *mp; // the forward's L and the reference of its sum (backward)
    // backward partials
    int nshares, layer;        // shares, blocks of a round over the compute units
    int64_t share;             // half-tiles per share, rounded down, and the rest
    int share_rem;
    int64_t nb, ntiles;        // 64-point blocks, tiles
    float *Zr;                 // per share and row of tiles it touches: K x 64 row-side partials
    float *Zc;                 // per tile, then per share: K x 64 column-side partials
    double *zpair;         // per short pair: a (y_i - y_j), K values
};

// (m1, s1) <- (m1, s1) merged with (m2, s2), FP64.
__device__ __forceinline__ void lse_merge(double &m1, double &s1, double m2, double s2, double tau) {
    if (!(s2 > 0.0)) return;
    if (!(s1 > 0.0)) { m1 = m2; s1 = s2; return; }
    const double m = fmin(m1, m2);
    s1 = s1 * exp((m - m1) / tau) + s2 * exp((m - m2) / tau);
    m1 = m;
}

// Block-wide merge of per-thread (m, s) into *out (thread 0).  All threads call.
__device__ void block_lse(double m, double s, double tau, SmPart *out) {
    __shared__ SmPart sp[kPairBlock / kWave];
#pragma unroll 1
    for (int o = 32; o > 0; o >>= 1) {
        const double m2 = __shfl_xor(m, o, kWave);
        const double s2 = __shfl_xor(s, o, kWave);
        lse_merge(m, s, m2, s2, tau);
    }
    if ((threadIdx.x & 63) == 0) sp[threadIdx.x >> 6] = SmPart{m, s};
    __syncthreads();
    if (threadIdx.x == 0) {
        double mm = sp[0].m, ss = sp[0].s;
        for (int w = 1; w < kPairBlock / kWave; ++w) lse_merge(mm, ss, sp[w].m, sp[w].s, tau);
        *out = SmPart{mm, ss};
    }
}

#ifndef SAP_KINST
// P (n x k row-major FP32) -> k x n FP64, and the copy that the backward's P
// is compared with.
__global__ void k_sm_loadP(const float *__restrict__ P, int n, int k, double *__restrict__ P64t,
                           float *__restrict__ P32) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n * k) return;
    const int l = e / k, q = e % k;
    const float v = P[e];
    P64t[(int64_t)q * n + l] = (double)v;
    P32[e] = v;
}

// Whether P is, bit for bit, the forward's P: for k_sm_dP and for the host
// (pinned memory).
constexpr int kSameBlock = 1024;
__global__ __launch_bounds__(kSameBlock) void k_sm_same(const float *__restrict__ P, const float *__restrict__ P32,
                                                        int nk, DevState *__restrict__ st,
                                                        int32_t *__restrict__ host) {
    int diff = 0;
    for (int e = threadIdx.x; e < nk; e += kSameBlock) diff |= __float_as_int(P[e]) != __float_as_int(P32[e]);
    diff = __syncthreads_or(diff);
    if (threadIdx.x == 0) {
        st->sm_same = !diff;
        *host = !diff;
    }
}

#endif

// Short pairs in FP64 (c = P^T (x_i - x_j) on the matrix cores, 16 pairs per
// wavefront, grid-stride).  Forward: the block's (min, sum) partial.
// Backward: a (y_i - y_j) = exp(-(r - L)/tau) / (r d^2) c per pair into zpair
// (lane m writes component m).
template <int K, typename TX>
__device__ void sm_short_block(const SmArgs &a, const TX *__restrict__ X, int64_t ldx, int sb,
                               int nshort, int bwd) {
    const int lane = threadIdx.x & 63;
    const int m = lane & 15, kk = lane >> 4;
    const int64_t ngroups = (a.nclose + 15) / 16;
    const double tau = a.tau;
    const double L = bwd ? *a.Lp : 0.0;
    double mm = 0.0, ss = 0.0;
    for (int64_t g16 = (int64_t)sb * (kPairBlock / kWave) + (threadIdx.x >> 6); g16 < ngroups;
         g16 += (int64_t)nshort * (kPairBlock / kWave)) {
        const int64_t row = g16 * 16 + m;
        const bool rin = row < a.nclose;
        const int2 pr = a.close[rin ? row : a.nclose - 1];
        const double dlen = a.cd[rin ? row : a.nclose - 1];
        const double4_t acc = short_c16<K, TX>(X, ldx, pr, rin, a.n, a.P64t, a.vx, a.vp);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const double q2 = row_sum16(acc[v] * acc[v]);
            const int src = kk + 4 * v;          // the lane (m = src) that loaded this pair
            const double d = __shfl(dlen, src, kWave);
            const int64_t e = g16 * 16 + src;
            if (e < a.nclose) {
                const double r = sqrt(q2) / d;
                if (!bwd) {
                    if (m == 0) lse_merge(mm, ss, r, 1.0, tau);
                } else if (m < K) {
                    const double coef = r > 0.0 ? exp(-(r - L) / tau) / (r * d * d) : 0.0;
                    a.zpair[e * K + m] = coef * acc[v];
                }
            }
        }
    }
    if (!bwd) block_lse(mm, ss, tau, a.part + a.npass + sb);
}

// Blocks below gemm_blocks: Y = (X - mu) P; the others: short pairs.
template <int K, typename TX>
__global__ __launch_bounds__(kPairBlock) void k_sm_prep(SmArgs a, const TX *__restrict__ X,
                                                        int64_t ldx, int64_t N,
                                                        const double *__restrict__ mu,
                                                        float *__restrict__ Y, int64_t Npad,
                                                        int gemm_blocks, int bwd) {
    if ((int)blockIdx.x < gemm_blocks)
    {
        const TX nx[16] = {};
        const double none[16] = {};
        gemm_block<TX>(X, ldx, N, a.n, K, mu, a.P64t, Y, nullptr, a.kp, Npad, a.vx, a.vp, nx, none, false,
                       a.gemm);
    }
    else
        sm_short_block<K, TX>(a, X, ldx, (int)blockIdx.x - gemm_blocks, (int)gridDim.x - gemm_blocks,
                              bwd);
}

__device__ __forceinline__ float comp4(const float4 &v, int r) {
    return r == 0 ? v.x : r == 1 ? v.y : r == 2 ? v.z : v.w;
}

// Forward pass: half-tiles dealt to the wavefronts of a resident grid (as the
// pair pass: y_i rows by scalar loads, the next half-tile's weights and y_j in
// flight during the current one).  Per lane, the 32 r of a half-tile are
// reduced to their min m_c and s_c = sum 2^((m_c - r) c2), then folded into
// the lane's running (m, s).  A masked pair's 1/d^2 is -1 or -2: its r is NaN
// (1/d^2 itself is added to its r^2, which alone would be -0 where y_i = y_j;
// for the others the addend is 0), which the minimum passes over and the
// clamp of its term to [0, 1] (a modifier of the exponential) makes 0.  A
// constant start of the sum of squares would do without the addend, but it is
// a length: next to coordinates of 1e-15 1e-36 is not small any more.
// Bound by VALU issue, 2K + 8 instructions per pair (142 us at N = 20000, k =
// 10 if sqrt and exp2 took one slot each): 157 to 172 us from card to card; 224
// with the y_i rows through LDS, 8192 blocks and an instruction more per
// pair.  N = 1531, k = 3: 6 us (10).
template <int K>
__global__ __launch_bounds__(kPairBlock, 4) void k_sm_fwd(SmArgs a) {
    constexpr int KP = K <= 4 ? 4 : (K <= 8 ? 8 : (K <= 12 ? 12 : 16));   // the Y row length (a.kp)
    constexpr int R = KP >= 12 ? 2 : KP == 8 ? 4 : 8;                     // y_i rows per scalar group
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t nw = (int64_t)a.npass * (kPairBlock / kWave);
    const float c2 = a.c2;
    float m = 1e30f;
    double s = 0.0;
    int64_t h = (int64_t)blockIdx.x * (kPairBlock / kWave) + wv;
    float4 w[8];
    float yj[K];
    int2 bt, btn;
    auto tile_of = [&](int64_t hh) __attribute__((always_inline)) {
        const int2_bits v = *(UniformI2)(a.tiles + ((hh < a.nhalf ? hh : a.nhalf - 1) >> 1));
        return make_int2(v.x, v.y);
    };
    auto weights = [&](int64_t hh) __attribute__((always_inline)) {
        return a.invd2 + (hh >> 1) * (kTileElems / 4) + (int)(hh & 1) * 512 + lane;
    };
    auto item = [&](auto pf) __attribute__((always_inline)) {
        constexpr bool PF = decltype(pf)::value;
        const UniformF yi0 = (UniformF)(a.Y + ((int64_t)bt.x * kTile + 32 * (int)(h & 1)) * KP);
        const float4 *wn = weights(h + nw);
        float yjn[K];
        if constexpr (PF) load_yj<K>(a.Y, KP, (int64_t)btn.y * kTile + lane, yjn);
        float r[32];
        float mc = 1e30f;
        float yr[2][R][KP];
        load_rows<KP, R>(yi0, yr[0]);
#pragma unroll
        for (int e0 = 0; e0 < 32; e0 += R) {
            wait_rows<KP, R>(yr[(e0 / R) & 1]);
            if (e0 + R < 32) load_rows<KP, R>(yi0 + (e0 + R) * KP, yr[(e0 / R + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int rr = 0; rr < R; ++rr) {
                const int e = e0 + rr;
                float acc = 0.0f;
#pragma unroll
                for (int c = 0; c < K; ++c) {
                    const float d = yr[(e0 / R) & 1][rr][c] - yj[c];
                    acc = __builtin_fmaf(d, d, acc);
                }
                const float wt = comp4(w[e / 4], e % 4);
                r[e] = __builtin_amdgcn_sqrtf(__builtin_fmaf(acc, wt, __builtin_amdgcn_fmed3f(wt, -2.0f, 0.0f)));
                asm volatile("" : "+v"(r[e]));   // computed here: deferred, the rows would outlive the scalar registers
                mc = fminf(mc, r[e]);
                if constexpr (PF)
                    if (e % 4 == 3) w[e / 4] = wn[(e / 4) * 64];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        float sc = 0.0f;
        const float mcc = mc * c2;
#pragma unroll
        for (int e = 0; e < 32; ++e)
            sc += __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(__builtin_fmaf(-r[e], c2, mcc)), 0.0f, 1.0f);
        const float mn = fminf(m, mc);
        s = s * (double)__builtin_amdgcn_exp2f((mn - m) * c2) +
            (double)(sc * __builtin_amdgcn_exp2f((mn - mc) * c2));
        m = mn;
        if constexpr (PF) {
#pragma unroll
            for (int c = 0; c < K; ++c) yj[c] = yjn[c];
        }
    };
    if (h < a.nhalf) {
        bt = tile_of(h);
        btn = tile_of(h + nw);
        const float4 *tp = weights(h);
#pragma unroll
        for (int g = 0; g < 8; ++g) w[g] = tp[g * 64];
        load_yj<K>(a.Y, KP, (int64_t)bt.y * kTile + lane, yj);
        for (; h + nw < a.nhalf; h += nw) {
            const int2 bt2 = tile_of(h + 2 * nw);
            item(std::true_type{});
            bt = btn;
            btn = bt2;
        }
        item(std::false_type{});
    }
    block_lse((double)m, s, a.tau, a.part + blockIdx.x);
}

#ifndef SAP_KINST
// Final merge of the forward (one block): L = m - tau log s.
__global__ __launch_bounds__(kPairBlock) void k_sm_fin(const SmPart *__restrict__ part, int nparts,
                                                       double tau, float *__restrict__ loss,
                                                       DevState *st) {
    double m = 0.0, s = 0.0;
    for (int b = threadIdx.x; b < nparts; b += kPairBlock) lse_merge(m, s, part[b].m, part[b].s, tau);
    __shared__ SmPart out;
    block_lse(m, s, tau, &out);
    __syncthreads();
    if (threadIdx.x == 0) {
        const double L = out.s > 0.0 ? out.m - tau * log(out.s) : __builtin_huge_val();
        st->sm_m = out.m;
        st->sm_s = out.s;
        st->sm_L = L;
        loss[0] = (float)L;
    }
}

#endif

// Row stride of a wavefront's 32 x 64 weight block in LDS.  66 = 2 mod 32
// words: the row contraction's reads (16 rows x 4 consecutive columns) meet
// every bank once per half-wavefront, and the phase-1 writes (one row, 64
// consecutive columns) too.
constexpr int kAStride = 66;

// First half-tile of share w (of a.nshares equal runs, to one half-tile).
__device__ __forceinline__ int64_t share_start(const SmArgs &a, int w) {
    return w * a.share + (unsigned)w * (unsigned)a.share_rem / (unsigned)a.nshares;
}

// The share that holds half-tile p: the last that starts at or before it.
__device__ __forceinline__ int share_of(const SmArgs &a, int64_t p) {
    int w = (int)((double)p * (double)a.nshares / (double)a.nhalf);
    while (w + 1 < a.nshares && share_start(a, w + 1) <= p) ++w;
    while (share_start(a, w) > p) --w;
    return w;
}

// Backward pass: one wavefront per share, a run of consecutive half-tiles (32
// rows of a tile), row of tiles by row of tiles.
// Phase 1 of a half-tile (lane = column j): the weights a_ij of the lane's
// column, one float4 of 1/d^2 per four rows (y_i rows by scalar loads), and
// the column side
//   z_j += sum_i a_ij (y_j - y_i)
// accumulated in FP32 from the differences y_i - y_j that the weight needed
// anyway, over the halves of the tile that the share holds, eight rows and
// then the eights: a sum over 64 rows in a row would round twice as often as
// one over a half-tile, this rounds a quarter as often.  a_ij goes to the
// wavefront's LDS block.
// Phase 2: the row side
//   z_i += sum_j a_ij (y_i - y_j) = (sum_j a_ij) y_i - (A Y_J)_i
// on the matrix cores in FP64 (v_mfma_f64_16x16x4f64, K padded to 16
// columns): lane (c16 = lane % 16, r4 = lane / 16) feeds A = a[16 mb + c16]
// [4 t + r4] from LDS and B = y_J[4 t + r4][c16].  The FP32 weights and
// coordinates are exact in FP64 and the products and sums FP64, so the
// difference of the two large terms keeps the accuracy of the direct sum of
// differences.  For K < 16 the padding column 15 of B is 1, which makes
// column 15 of the product the row sum; K = 16 sums the rows separately.  The
// products accumulate over a row of tiles, and the row side is formed at its end.
//
// Partials, component-major in FP32: Zr once per row, Zc once per tile, and
// once more for a tile whose halves fall in two shares.  Per half-tile and
// point-major they were 377 MB written and read again at N = 20000, k = 10
// (k_sm_zred 90 us, 32 now, traced).
// Bound by issue: 3K + 8 VALU instructions per pair, K/8 for the sums by eights,
// a sixth more around the products, and the FP64 products, which other wavefronts' VALU work covers in
// part: N = 20000, k = 10 383 us (407 with a block per half-tile and the rows
// through LDS), N = 14000, k = 16 250 (296), N = 9000, k = 10 85 (79: the merge
// gained what this lost, 6 us).
// LDS per block: 37 KB (K <= 4) to 49 KB (K >= 13): three blocks per compute
// unit, two for K >= 13 (at three they would spill).
template <int K>
__global__ __launch_bounds__(kPairBlock, K <= 12 ? 3 : 2) void k_sm_bwd(SmArgs a) {
    constexpr int KP = K <= 4 ? 4 : (K <= 8 ? 8 : (K <= 12 ? 12 : 16));   // the Y row length (a.kp)
    __shared__ float4 s_yc[kPairBlock / kWave][64 * KP / 4];
    __shared__ float s_a[kPairBlock / kWave][32 * kAStride];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float c2 = a.c2;
    const float Lc = (float)(*a.Lp) * c2;
    float4 *ycl = s_yc[wv];
    float *al = s_a[wv];
    const float *yc0 = reinterpret_cast<const float *>(ycl);
    const int c16 = lane & 15, r4 = lane >> 4;
    const bool qin = c16 < K;
    const int qc = qin ? c16 : K - 1;                 // clamped component: in-bounds reads
    const double bpad = (K < 16 && c16 == 15) ? 1.0 : 0.0;
    const float *alr = al + c16 * kAStride + r4;      // row-side reads: + 16 mb kAStride + 4 u
    // the shares that one SIMD gets (blocks c, c + layer, ..., same wavefront)
    // are neighbours: their lengths add to the same total, to one half-tile
    const int w = (((int)blockIdx.x % a.layer) * (kPairBlock / kWave) + wv) * (a.nshares / (a.layer * (kPairBlock / kWave))) +
                  (int)blockIdx.x / a.layer;
    int64_t p = share_start(a, w);
    const int64_t p1 = share_start(a, w + 1);
    int bi = ((UniformI2)(a.tiles + (p >> 1)))->x;
    do {                                              // (an empty share: a row side of zeros)
        const int64_t trow = (int64_t)bi * a.nb - (int64_t)bi * (bi - 1) / 2;   // tile (bi, bi)
        const int64_t row1 = 2 * (trow + a.nb - bi);
        const int h0 = (int)(p - 2 * trow), h1 = (int)((p1 < row1 ? p1 : row1) - 2 * trow);
        const float4 *trow4 = a.invd2 + trow * (kTileElems / 4) + lane;
        const float *yrow = a.Y + (int64_t)bi * kTile * KP;
        auto column = [&](int h) __attribute__((always_inline)) {
            return reinterpret_cast<const float4 *>(a.Y + ((int64_t)(bi + (h >> 1)) * kTile + lane) * KP);
        };
        double4_t accr[4];
        double rs[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) { accr[u] = double4_t{0.0, 0.0, 0.0, 0.0}; rs[u] = 0.0; }
        // the first tile's column rows and the first weights
        float4 yv[KP / 4], wq[2];
#pragma unroll
        for (int u = 0; u < KP / 4; ++u) yv[u] = column(h0)[u];
        wq[0] = trow4[(int64_t)h0 * 512];
        wq[1] = trow4[(int64_t)h0 * 512 + 64];
        for (int h = h0; h < h1;) {
            float yj[K], zc[K];
            __builtin_amdgcn_wave_barrier();   // (the previous tile's columns have been read)
#pragma unroll
            for (int u = 0; u < KP / 4; ++u) ycl[lane * (KP / 4) + u] = yv[u];
#pragma unroll
            for (int q = 0; q < K; ++q) {
                yj[q] = comp4(yv[q / 4], q % 4);
                zc[q] = 0.0f;
            }
            const int hn = (h | 1) + 1;        // the next tile's first half
            {   // its column rows (this tile's again at the end)
                const float4 *src = column(hn < h1 ? hn : h);
#pragma unroll
                for (int u = 0; u < KP / 4; ++u) yv[u] = src[u];
            }
            auto half_tile = [&](auto hsel) __attribute__((always_inline)) {
                constexpr int HS = decltype(hsel)::value;
                const float4 *tp = trow4 + (int64_t)h * 512;
                const float4 *tpn = trow4 + (int64_t)(h + 1 < h1 ? h + 1 : h) * 512;
                const UniformF yi0 = (UniformF)(yrow + 32 * HS * KP);
#pragma unroll 1
                for (int g = 0; g < 8; g += 2) {
                    float z8[K];   // the column side of these eight rows
#pragma unroll
                    for (int g2 = 0; g2 < 2; ++g2) {
                        const float4 w4 = wq[g2];
                        wq[g2] = g < 6 ? tp[(g + 2 + g2) * 64] : tpn[g2 * 64];
                        float yr[4][KP];
                        load_rows<KP, 4>(yi0 + 4 * (g + g2) * KP, yr);
#pragma unroll
                        for (int rr = 0; rr < 4; ++rr) {
                            const float wt = comp4(w4, rr);
                            float d[K];
                            float acc2 = 0.0f;
#pragma unroll
                            for (int q = 0; q < K; ++q) {
                                d[q] = yr[rr][q] - yj[q];
                                acc2 = __builtin_fmaf(d[q], d[q], acc2);
                            }
                            // masked pairs (1/d^2 < 0) and r = 0: the reciprocal
                            // root makes NaN of both, the maximum 0 of that
                            const float r2 = acc2 * wt;
                            const float rinv = __builtin_amdgcn_rsqf(r2);
                            const float rv = r2 * rinv;
                            const float ex = __builtin_amdgcn_exp2f(__builtin_fmaf(-rv, c2, Lc));
                            const float av = fmaxf(ex * wt * rinv, 0.0f);
#pragma unroll
                            for (int q = 0; q < K; ++q)
                                z8[q] = g2 + rr == 0 ? -av * d[q] : __builtin_fmaf(-av, d[q], z8[q]);
                            al[(4 * (g + g2) + rr) * kAStride + lane] = av;
                        }
                    }
#pragma unroll
                    for (int q = 0; q < K; ++q) zc[q] += z8[q];
                }
                __builtin_amdgcn_wave_barrier();
                // phase 2: A[16 mb + c16][4 u + r4] from LDS, B = Y_J[4 u + r4][c16]
#pragma unroll 4
                for (int u = 0; u < 16; ++u) {
                    const int jc = 4 * u + r4;
                    const float yv2 = yc0[jc * KP + qc];
                    const double bq = qin ? (double)yv2 : bpad;
                    const double a0 = (double)alr[4 * u];
                    const double a1 = (double)alr[16 * kAStride + 4 * u];
                    if constexpr (K == 16) {
                        rs[2 * HS] += a0;
                        rs[2 * HS + 1] += a1;
                    }
                    accr[2 * HS] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, bq, accr[2 * HS], 0, 0, 0);
                    accr[2 * HS + 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, bq, accr[2 * HS + 1], 0, 0, 0);
                }
                __builtin_amdgcn_wave_barrier();
                ++h;
            };
            const bool tail = h & 1;           // the tile's first half lies in the share before
            float *zcol = a.Zc + (tail ? a.ntiles + w : trow + (h >> 1)) * (int64_t)(K * 64) + lane;
            if (!tail) half_tile(std::integral_constant<int, 0>{});
            if (h < hn && h < h1) half_tile(std::integral_constant<int, 1>{});
#pragma unroll
            for (int q = 0; q < K; ++q) zcol[q * 64] = zc[q];
        }
        float *zrow = a.Zr + (w + bi) * (int64_t)(K * 64);
        // lane holds (A Y_J)[16 mb + r4 + 4 v][c16]; row (r4 + 4 v)'s sum sits
        // in the lanes with c16 = r4 + 4 v (K = 16), or in column 15 of the
        // product, lane (r4, 15) (K < 16)
#pragma unroll
        for (int mb = 0; mb < 4; ++mb) {
            if constexpr (K == 16) {
                rs[mb] += __shfl_xor(rs[mb], 16, kWave);
                rs[mb] += __shfl_xor(rs[mb], 32, kWave);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = 16 * mb + r4 + 4 * v;
                double sm;
                if constexpr (K == 16) sm = __shfl(rs[mb], (lane & 48) | (r4 + 4 * v), kWave);
                else sm = __shfl(accr[mb][v], (lane & 48) | 15, kWave);
                const double z = sm * (double)yrow[(int64_t)i * KP + qc] - accr[mb][v];
                if (qin) zrow[c16 * 64 + i] = (float)z;
            }
        }
        p = row1;
        ++bi;
    } while (p < p1);
}

// z_p for the 64 points of point block b (one block of eight wavefronts per
// point block): row-side partials of the items of row b, column-side partials
// of tiles (bi <= b, b), then the short pairs through their CSR segments
// (pairs with i = p add, pairs with j = p subtract).  The wavefronts split the
// terms; their sums are added in a fixed order.
constexpr int kZredWaves = 8;
template <int K>
__global__ __launch_bounds__(kZredWaves * kWave) void k_sm_zred(SmArgs a, int64_t nb, int64_t N,
                                                                const int32_t *__restrict__ rp_i,
                                                                const int32_t *__restrict__ rp_j,
                                                                const int32_t *__restrict__ permj,
                                                                double *__restrict__ Z) {
    __shared__ double sz[kZredWaves][64 * K];
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int64_t b = blockIdx.x;
    double z[K];
#pragma unroll
    for (int q = 0; q < K; ++q) z[q] = 0.0;
    // two partials per step, all their loads issued before the adds
    auto add2 = [&](const float *z0, const float *z1) __attribute__((always_inline)) {
        float u0[K], u1[K];
#pragma unroll
        for (int q = 0; q < K; ++q) { u0[q] = z0[q * 64]; u1[q] = z1[q * 64]; }
#pragma unroll
        for (int q = 0; q < K; ++q) z[q] += (double)u0[q] + (double)u1[q];
    };
    auto add1 = [&](const float *z0) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < K; ++q) z[q] += (double)z0[q * 64];
    };
    const int64_t len = K * 64;
    // rows: the shares that touch row b
    const int64_t trow = b * nb - b * (b - 1) / 2;
    const int64_t i1 = share_of(a, 2 * (trow + nb - b) - 1) + b;
    int64_t ix = share_of(a, 2 * trow) + b + wv;
    for (; ix + kZredWaves <= i1; ix += 2 * kZredWaves)
        add2(a.Zr + ix * len + lane, a.Zr + (ix + kZredWaves) * len + lane);
    if (ix <= i1) add1(a.Zr + ix * len + lane);
    // columns: the tiles (bi, b), then the second halves in shares of their own
    auto col = [&](int64_t bi) { return a.Zc + (bi * nb - bi * (bi - 1) / 2 + (b - bi)) * len + lane; };
    int64_t bi = wv;
    for (; bi + kZredWaves <= b; bi += 2 * kZredWaves) add2(col(bi), col(bi + kZredWaves));
    if (bi <= b) add1(col(bi));
    for (int64_t b0 = wv; b0 <= b; b0 += kZredWaves * kWave) {   // (a lane per tile)
        bi = b0 + kZredWaves * lane;
        const int64_t x = 2 * (bi * nb - bi * (bi - 1) / 2 + (b - bi)) + 1;
        const int w = bi <= b ? share_of(a, x) : 0;
        for (uint64_t hit = __ballot(bi <= b && share_start(a, w) == x); hit; hit &= hit - 1)
            add1(a.Zc + (a.ntiles + __shfl(w, __ffsll((unsigned long long)hit) - 1, kWave)) * len + lane);
    }
    // the tile weights were taken at L c2 rounded to FP32, and c2 itself is
    // rounded: what that took from their exponent, the same for every pair, is
    // put back here (the short pairs' weights are FP64).  The weights sum to 1
    // when L - m (m the reference of the forward's sum, the r that count are
    // near it) takes the exact c2 and m, as r, the rounded one: with L c2 the
    // gradient was off by (m - L) / tau times c2's rounding, 2e-7 to 5e-7 of it
    // where tau is 0.3.
    const double L = *a.Lp, m = *a.mp;
    const double corr = exp2(m * (double)a.c2 + (L - m) * a.c2d - (double)((float)L * a.c2));
#pragma unroll
    for (int q = 0; q < K; ++q) z[q] *= corr;
    const int64_t p = b * kTile + lane;
    if (a.nclose > 0 && p < N) {
        for (int32_t e = rp_i[p] + wv; e < rp_i[p + 1]; e += kZredWaves) {
#pragma unroll
            for (int q = 0; q < K; ++q) z[q] += a.zpair[(int64_t)e * K + q];
        }
        for (int32_t e = rp_j[p] + wv; e < rp_j[p + 1]; e += kZredWaves) {
            const int64_t ee = permj[e];
#pragma unroll
            for (int q = 0; q < K; ++q) z[q] -= a.zpair[ee * K + q];
        }
    }
#pragma unroll
    for (int q = 0; q < K; ++q) sz[wv][lane * K + q] = z[q];
    __syncthreads();
    for (int e = threadIdx.x; e < 64 * K; e += kZredWaves * kWave) {
        if (b * kTile + e / K < N) {
            double acc = 0.0;
#pragma unroll
            for (int w = 0; w < kZredWaves; ++w) acc += sz[w][e];
            Z[b * kTile * K + e] = acc;
        }
    }
}

#ifndef SAP_KINST
// G_c = sum_{p in chunk c} (x_p - mu) z_p^T (n x K, element e = q n + l) on
// the matrix cores in FP64 (v_mfma_f64_16x16x4f64): output rows are 16
// components l of x, the contraction runs over the chunk's points four at a
// time.  Lane (c16, r4) feeds A = x[p][16 mb + c16] - mu and B = z[p][c16]
// for p = p0 + 4 s + r4; wavefront w takes the component blocks mb = w,
// w + 4, ...  Rows past the chunk and columns past n or K contribute 0
// (selects, not multiplies, so no value of a masked element matters).
template <typename TX>
__global__ __launch_bounds__(256) void k_sm_grad(const TX *__restrict__ X, int64_t ldx, int64_t N,
                                                 int n, int K, const double *__restrict__ mu,
                                                 const double *__restrict__ Z, int64_t rows,
                                                 double *__restrict__ Gpart) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int c16 = lane & 15, r4 = lane >> 4;
    const int64_t p0 = (int64_t)blockIdx.x * rows;
    const int64_t p1 = p0 + rows < N ? p0 + rows : N;
    const int64_t nsteps = (p1 - p0 + 3) / 4;
    const int nmb = (n + 15) / 16;
    const bool qin = c16 < K;
    const int qc = qin ? c16 : K - 1;
    double *out = Gpart + (int64_t)blockIdx.x * n * K;
    for (int mb = wv; mb < nmb; mb += 4) {
        const int l = 16 * mb + c16;
        const bool lin = l < n;
        const int lc = lin ? l : n - 1;
        const double ml = mu[lc];
        double4_t acc = {0.0, 0.0, 0.0, 0.0};
        for (int64_t s0 = 0; s0 < nsteps; s0 += 4) {
            double xa[4], zb[4];
            bool pin[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t p = p0 + 4 * (s0 + u) + r4;
                pin[u] = p < p1;
                const int64_t pc = pin[u] ? p : p0;
                xa[u] = (double)X[pc * ldx + lc];
                zb[u] = Z[pc * K + qc];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const double av = (pin[u] && lin) ? xa[u] - ml : 0.0;
                const double bv = (pin[u] && qin) ? zb[u] : 0.0;
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
            }
        }
        // lane holds G[16 mb + r4 + 4 v][c16]
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int lo = 16 * mb + r4 + 4 * v;
            if (lo < n && qin) out[(int64_t)c16 * n + lo] = acc[v];
        }
    }
}

// dP (n x k row-major FP32) = dL/dloss * sum over the chunks: one block per
// 64 output elements; its four wavefronts take every fourth chunk, with
// eight loads in flight per lane, and their sums are added in a fixed order.
__global__ __launch_bounds__(256) void k_sm_dP(const double *__restrict__ Gpart, int nchunks, int n,
                                               int K, const float *__restrict__ grad_loss,
                                               float *__restrict__ dP, const DevState *__restrict__ st) {
    if (!st->sm_same) return;
    __shared__ double sp[4][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + lane;
    const int nk = n * K;
    double acc = 0.0;
    if (e < nk) {
        int c = wv;
        for (; c + 28 < nchunks; c += 32) {
            double t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = Gpart[(int64_t)(c + 4 * u) * nk + e];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc += t[u];
        }
        for (; c < nchunks; c += 4) acc += Gpart[(int64_t)c * nk + e];
    }
    sp[wv][lane] = acc;
    __syncthreads();
    if (wv == 0 && e < nk) {
        const int l = e % n, q = e / n;
        const double g = ((sp[0][lane] + sp[1][lane]) + sp[2][lane]) + sp[3][lane];
        dP[(int64_t)l * K + q] = (float)((double)grad_loss[0] * g);
    }
}

#endif

}  // namespace sap
