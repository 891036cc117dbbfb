// Batched SAP (gfx950): many independent small problems, Algorithm 1 (Sec. 4)
// on all of them side by side.
//
// The paper applies Algorithm 1 to many small secant sets: for every target
// dimension of a sweep (Sec. 6.1), to random subsamples of a data set whose
// full secant matrix does not fit (Sec. 6.3), and with the length threshold
// of Sec. 7.  An iteration is two launches for the whole batch, each problem
// with its own blocks in both (the kernel boundary is the barrier between
// them, as in the single-problem run):
//   pass       every 16 x 64 quarter of the set's 64 x 64 tiles: ||y_i - y_j||^2
//              (FP64 differences) times the stored FP32 1/d^2, rounded to an
//              FP32 key; the candidate window of the block's running minimum,
//              as in the single-problem pass; then the block's window pairs in
//              FP64 from X (the same routine), one result per block;
//   selection  every block of a problem takes the lexicographic (r, i, j)
//              minimum of the problem's results and applies the FP64 argmax /
//              modified Gram-Schmidt / shift of the single-problem handle in
//              LDS, then computes its rows of Y = (X_S - mean_S) P' in FP64 on
//              the matrix cores (v_mfma_f64_16x16x4f64), the set's rows gathered
//              through its index list; the problem's first block writes the
//              trace entry and P'.
// One workgroup per problem for the whole run -- no launches between the
// phases, but 4 wavefronts on one compute unit -- took 52 us per iteration at
// 30 problems of 256 points (n = 15) and 184 us at 60 of 512 points (n =
// 200), against 21 and 43 us.  Batches whose sets are all small enough run that
// way (k_batch_run; one_block_per_problem draws the line), and batches whose
// two-launch buffers do not fit the fixed scratch.
//
// Y stays FP64, so the coarse error is that of the FP64 product (no pair is
// too short for it and there is no short-pair list); keys round to FP32.
//
// Scratch (device): per-set index lists, tile tables and 1/d^2 tiles (FP32,
// the single-problem layout), per-set mean / radius / largest kept 1/d^2 /
// pair counts, per-problem P (kp x n FP64, rows >= k zero) and Y (Mpad x kp
// FP64); for the two launches P twice (the selection reads one and writes the
// other), block tables and block results.
#define SAP_KINST 1

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <limits>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include <hip/hip_ext.h>

#include "sap_dist.h"
#include "sap_iter.hip"
#include "sap_mem.h"

namespace sap {

constexpr int kBatchMaxPoints = 32768;
constexpr int kBatchLdsDoubles = 16384;   // the update's (k + 2) n doubles: 128 KB beside the pass's 31 KB

struct BatchSet {        // per point set
    int64_t pt_off;      // first entry of its row-index list
    int64_t tile_off;    // first tile (tile table and 1/d^2 tiles)
    int32_t M, nb;       // points, 64-point blocks
    int32_t ntiles, pad;
};

struct BatchProb {       // per problem
    int32_t set, k, kp, rule;
    double alpha;
    int64_t P_off;       // its kp x n P in Pbuf (doubles)
    int64_t Y_off;       // its Mpad x kp Y in Ybuf (doubles)
    int64_t P0_off;      // its n x k block in the caller's P0 / P_out (doubles)
};

// per-set statistics written by the precomputation
struct BatchStat {
    uint64_t radius_bits;   // max ||x - mean|| (FP64 bits; non-negative)
    uint32_t wmax_bits;     // largest FP32 1/d^2 of a kept pair (bits)
    int32_t nonfinite;
    uint64_t kept, dropped;
};

// What the blocks of the run need of a problem and its set, in one record:
// npass blocks of the pass (their results at part_off), and selection blocks
// of 64 gt rows of Y each.
struct BatchDesc {
    int64_t pt_off, tile_off, P_off, Y_off, part_off;
    double alpha;
    int32_t set, k, kp, rule;
    int32_t M, nb, ntiles;
    int32_t npass, gt, pad;
};

// The record of a problem with one block.
__host__ __device__ inline BatchDesc batch_desc(const BatchProb &p, const BatchSet &st) {
    return BatchDesc{st.pt_off, st.tile_off, p.P_off, p.Y_off, 0, p.alpha, p.set, p.k, p.kp, p.rule,
                     st.M, st.nb, st.ntiles, 1, 1, 0};
}

// a start's check: max |P^T P - I| and whether an entry is NaN or Inf
struct BatchCheck {
    double err;
    int32_t nonfinite, pad;
};

struct BatchArgs {
    const void *X;
    int64_t ldx;
    int n, vx;
    const int32_t *pts;
    const BatchSet *sets;
    const BatchProb *probs;
    const int4 *tiles;       // (bi, bj, set, 0) per tile
    float4 *w;               // 1/d^2 tiles (kTileElems floats each)
    double *mu;              // n_sets x n
    BatchStat *stat;         // n_sets
    const double *set_min_len;
    const BatchDesc *desc;
    BatchCheck *chk;
    const int2 *pass_blk, *sel_blk;   // (problem, block of it) per block of the two launches
    Partial *part;
    double *Pbuf, *Pnext;    // the current P of every problem and the next
    double *Ybuf;
    const double *P0;
    double *P_out;
    int iters, cap;
    double *tr_min;
    int64_t *tr_ij;
    int32_t *tr_cert;
};

// ---------------------------------------------------------------- precomputation

// zero the per-set statistics (a fill kernel, not a memset)
__global__ void k_batch_clear(BatchStat *stat, int n_sets) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s < n_sets) stat[s] = BatchStat{0ull, 0u, 0, 0ull, 0ull};
}

// mean of each set's rows, column by column in point order; flags NaN / Inf
template <typename TX>
__global__ __launch_bounds__(256) void k_batch_mean(BatchArgs a) {
    const int s = blockIdx.y;
    const int l = blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= a.n) return;
    const BatchSet st = a.sets[s];
    const TX *X = static_cast<const TX *>(a.X);
    double acc = 0.0;
    int bad = 0, p = 0;
    for (; p + 16 <= st.M; p += 16) {   // 16 rows' loads in flight, the sum in point order
        TX v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = X[(int64_t)a.pts[st.pt_off + p + u] * a.ldx + l];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            if (!isfinite(v[u])) bad = 1;
            acc += (double)v[u];
        }
    }
    for (; p < st.M; ++p) {
        const double v = (double)X[(int64_t)a.pts[st.pt_off + p] * a.ldx + l];
        if (!isfinite(v)) bad = 1;
        acc += v;
    }
    a.mu[(int64_t)s * a.n + l] = acc / (double)st.M;
    if (bad) atomicOr(&a.stat[s].nonfinite, 1);
}

// radius of each set: one wavefront per point
template <typename TX>
__global__ __launch_bounds__(256) void k_batch_radius(BatchArgs a) {
    const int s = blockIdx.y;
    const BatchSet st = a.sets[s];
    const int p = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (p >= st.M) return;
    const int lane = threadIdx.x & 63;
    const TX *x = static_cast<const TX *>(a.X) + (int64_t)a.pts[st.pt_off + p] * a.ldx;
    const double *mu = a.mu + (int64_t)s * a.n;
    double acc = 0.0;
    for (int l = lane; l < a.n; l += kWave) {
        const double t = (double)x[l] - mu[l];
        acc += t * t;
    }
    acc = wave_sum(acc);
    if (lane == 0) atomicMax(reinterpret_cast<unsigned long long *>(&a.stat[s].radius_bits),
                             (unsigned long long)__double_as_longlong(sqrt(acc)));
}

// 1/d^2 tiles of every set, by direct FP64 differences of the gathered rows
// (tile_dist2; the single-problem layout: element (r, c) of a tile at float
// index (r/4)*256 + c*4 + r%4).  Dropped pairs (duplicates, d < the set's l)
// and padding / i >= j hold -1.  Counts kept and dropped pairs per set and
// folds the largest kept FP32 value into the set's statistics.
template <typename TX>
__global__ __launch_bounds__(256, 4) void k_batch_invd2(BatchArgs a, int64_t ntiles_all) {
    __shared__ __align__(16) DistLds L;
    __shared__ unsigned s_kept, s_drop, s_wmax;
    const int ty = threadIdx.x >> 4, tx = threadIdx.x & 15;
    const TX *X = static_cast<const TX *>(a.X);
    for (int64_t t = blockIdx.x; t < ntiles_all; t += gridDim.x) {
        const int4 tb = a.tiles[t];
        const BatchSet st = a.sets[tb.z];
        const double ml = a.set_min_len ? a.set_min_len[tb.z] : 0.0;
        if (threadIdx.x == 0) { s_kept = 0u; s_drop = 0u; s_wmax = 0u; }
        if (threadIdx.x < 2 * kTile) {
            const int p = (threadIdx.x < kTile ? tb.x : tb.y) * kTile + (threadIdx.x & (kTile - 1));
            L.row[threadIdx.x] = a.pts[st.pt_off + (p < st.M ? p : st.M - 1)];
        }
        __syncthreads();
        double d2[4][4];
        tile_dist2(X, a.ldx, a.n, L, d2);
        const int i0 = tb.x * kTile + 4 * ty, j0 = tb.y * kTile;
        unsigned mx = 0u, nkept = 0u, ndrop = 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int j = j0 + tile_col(tx, q);
            float out[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = i0 + r;
                const double s = d2[r][q];
                float v = kMaskDropped;
                if (j < st.M && i < j) {
                    if (s == 0.0 || (ml > 0.0 && tile_shorter(X + (int64_t)L.row[i - tb.x * kTile] * a.ldx,
                                                              X + (int64_t)L.row[kTile + j - tb.y * kTile] * a.ldx,
                                                              a.n, s, ml))) {
                        ++ndrop;
                    } else {
                        v = (float)(1.0 / s);
                        ++nkept;
                        mx = max(mx, __float_as_uint(v));
                    }
                }
                out[r] = v;
            }
            a.w[t * (kTileElems / 4) + ty * 64 + tile_col(tx, q)] = make_float4(out[0], out[1], out[2], out[3]);
        }
        atomicAdd(&s_kept, nkept);
        atomicAdd(&s_drop, ndrop);
        atomicMax(&s_wmax, mx);
        __syncthreads();
        if (threadIdx.x == 0) {
            BatchStat *so = a.stat + tb.z;
            if (s_kept) atomicAdd(reinterpret_cast<unsigned long long *>(&so->kept), (unsigned long long)s_kept);
            if (s_drop) atomicAdd(reinterpret_cast<unsigned long long *>(&so->dropped), (unsigned long long)s_drop);
            if (s_wmax) atomicMax(&so->wmax_bits, s_wmax);
        }
        __syncthreads();
    }
}

// P0 blocks (n x k row-major) -> per-problem P (kp x n, rows >= k zero), every buffer
__global__ void k_batch_loadP(BatchArgs a) {
    const BatchProb pr = a.probs[blockIdx.y];
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    const int n = a.n;
    if (e >= pr.kp * n) return;
    const int q = e / n, l = e % n;
    const double v = q < pr.k ? a.P0[pr.P0_off + (int64_t)l * pr.k + q] : 0.0;
    a.Pbuf[pr.P_off + e] = v;
    if (a.Pnext) a.Pnext[pr.P_off + e] = v;   // (its rows >= k stay zero)
}

// The starts: one block per problem, entry (x, y) of P0^T P0 per thread, the
// rows in order and 16 at a time in flight (on the host, after a copy of every
// start, this took as long as ten iterations of 60 problems at n = 200).
__global__ __launch_bounds__(256) void k_batch_checkP(BatchArgs a) {
    __shared__ unsigned long long s_err;
    __shared__ int s_bad;
    const BatchProb pr = a.probs[blockIdx.x];
    const double *P = a.P0 + pr.P0_off;
    const int n = a.n, k = pr.k;
    if (threadIdx.x == 0) { s_err = 0ull; s_bad = 0; }
    __syncthreads();
    int bad = 0;
    for (int e = threadIdx.x; e < n * k; e += 256) bad |= isfinite(P[e]) ? 0 : 1;
    if (bad) atomicOr(&s_bad, 1);
    if ((int)threadIdx.x < k * k) {
        const int x = threadIdx.x / k, y = threadIdx.x % k;
        double acc = 0.0;
        int l = 0;
        for (; l + 16 <= n; l += 16) {
            double u[16], v[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) { u[q] = P[(l + q) * k + x]; v[q] = P[(l + q) * k + y]; }
#pragma unroll
            for (int q = 0; q < 16; ++q) acc += u[q] * v[q];
        }
        for (; l < n; ++l) acc += P[l * k + x] * P[l * k + y];
        const double e = fabs(acc - (x == y ? 1.0 : 0.0));
        // (a NaN ranks above inf by its bits: inf - inf off the diagonal stays
        // out, an infinite square of a column is on it)
        if (e >= 0.0) atomicMax(&s_err, (unsigned long long)__double_as_longlong(e));
    }
    __syncthreads();
    if (threadIdx.x == 0) a.chk[blockIdx.x] = BatchCheck{__longlong_as_double((long long)s_err), s_bad, 0};
}

// per-problem P (kp x n) -> P_out blocks (n x k row-major)
__global__ void k_batch_storeP(BatchArgs a) {
    const BatchProb pr = a.probs[blockIdx.y];
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= pr.k * a.n) return;
    const int l = e / pr.k, q = e % pr.k;
    a.P_out[pr.P0_off + e] = a.Pbuf[pr.P_off + (int64_t)q * a.n + l];
}

// ---------------------------------------------------------------- the run

// 16 rows of Y = (X_S - mean) P in FP64 (rows row0 .. row0 + 15 of the set;
// rows >= M are zero), kp columns (zero past the k rows of P, k x n): gemm16
// on rows gathered through the set's index list.
template <typename TX>
__device__ __forceinline__ void batch_gemm16(const TX *__restrict__ X, int64_t ldx, const int32_t *__restrict__ idx,
                                             int M, int n, int k, int kp, const double *__restrict__ mu,
                                             const double *P, double *__restrict__ Y, int row0, bool vx, bool vp) {
    const int lane = threadIdx.x & 63;
    const int m = lane & 15, kk = lane >> 4;
    const int row = row0 + m;
    const bool rin = row < M;
    const TX nx[16] = {};
    const double none[16] = {};
    const double4_t acc = gemm16<TX>(X + (int64_t)idx[rin ? row : M - 1] * ldx, rin, mu, P + (m < k ? m : k - 1) * n,
                                     m < k, n, vx, vp, nx, none, false);
    if (m < kp) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = row0 + kk + 4 * v;
            Y[(int64_t)r * kp + m] = r < M ? acc[v] : 0.0;
        }
    }
}

// The FP64 update of Algorithm 1 for the exact k (K_LO <= k <= K_HI), with
// P (k x n) staged in LDS, updated there and written to Pn (k x n, may be
// null): the single-problem handle's routines -- one wavefront with the
// vectors in registers when n <= 64 and k <= 8, the whole block over LDS
// otherwise.  Every thread of the block calls it.
template <typename TX, int K_LO, int K_HI>
__device__ __forceinline__ void batch_update(const TX *X, int64_t ldx, int n, int k, double *Pn, double alpha, int rule,
                                             int64_t gi, int64_t gj, double *sm) {
    if constexpr (K_LO <= K_HI) {
        if (k == K_LO) {
            if (K_LO <= 8 && n <= kWave) {
                if (threadIdx.x < kWave)
                    apply_update_reg<K_LO, 1, TX>(X, ldx, n, sm, Pn, nullptr, 0, alpha, rule, nullptr, gi, gj, true);
            } else {
                apply_update<K_LO, TX>(X, ldx, n, Pn, nullptr, 0, alpha, rule, nullptr, gi, gj, sm);
            }
        } else {
            batch_update<TX, K_LO + 1, K_HI>(X, ldx, n, k, Pn, alpha, rule, gi, gj, sm);
        }
    }
}

// LDS of a pass block, declared once in the kernel (the five KP variants
// share it): every wavefront's staged y_i rows and candidate list, the list
// lengths and the block's running minimum.
struct BatchLds {
    double y[kPairBlock / kWave][16 * kMaxK];
    int2 cij[kPairBlock / kWave][kCandCap];
    uint32_t ckey[kPairBlock / kWave][kCandCap];
    int cn[kPairBlock / kWave];
    uint32_t run;
};

// Tile (bi, bj), bi <= bj, of index t in the row-major order of a set's
// nb x nb upper triangle (t = bi nb - bi (bi - 1) / 2 + bj - bi): bi from the
// quadratic, corrected by at most a step each way.  Wavefront-uniform.
__device__ __forceinline__ int2 tile_of_index(int64_t t, int nb) {
    auto start = [nb](int64_t b) { return b * nb - b * (b - 1) / 2; };
    const double q = 2.0 * nb + 1.0;
    int64_t bi = (int64_t)floor((q - sqrt(fmax(q * q - 8.0 * (double)t, 0.0))) * 0.5);
    bi = bi < 0 ? 0 : (bi > nb - 1 ? nb - 1 : bi);
    while (bi > 0 && start(bi) > t) --bi;
    while (bi + 1 < nb && start(bi + 1) <= t) ++bi;
    return make_int2((int)bi, (int)(bi + (t - start(bi))));
}

// Coarse error bound of a problem's keys, |r~ - r| <= e_abs + e_rel r -- the
// FP64 product's error on y (norm over the k columns) and the FP32 rounding
// of 1/d^2 and of the key -- and item_window's coefficients.
struct BatchBound {
    double e_abs, e_rel;
    float wa, wb;
};
__device__ __forceinline__ BatchBound batch_bound(const BatchStat &bs, int n, int k, int kp) {
    BatchBound o;
    const double R = __longlong_as_double((long long)bs.radius_bits);
    const double delta = R * (double)(n + 2) * sqrt((double)k) * 1.1102230246251565e-16 * 4.0;
    const double wmax = (double)__uint_as_float(bs.wmax_bits);
    o.e_abs = bs.wmax_bits ? 2.0 * delta * sqrt(wmax * (1.0 + 2.384185791015625e-07)) : 0.0;
    o.e_rel = 2.0 * 5.9604644775390625e-08 + (kp + 4) * 1.1102230246251565e-16;
    o.wa = __uint_as_float(__float_as_uint((float)((1.0 + o.e_rel) / (1.0 - o.e_rel))) + 1u);
    o.wb = __uint_as_float(__float_as_uint((float)(2.0 * o.e_abs / (1.0 - o.e_rel))) + 1u);
    return o;
}

// Pass block lb of a problem: wavefront w takes the quarter tiles 4 lb + w, +
// 4 npass, ... (every load of an item is independent: tile coordinates are
// computed, not loaded), then the block's wavefronts share the rescoring of
// its window pairs.  PF: the next item's loads are issued before the current
// one's arithmetic, for a block that is alone on its compute unit (with the
// other blocks of a pass they would only cost registers).  Every thread of
// the block calls it and gets the result.
template <int KP, bool PF, typename TX>
__device__ __forceinline__ Partial batch_pass_block(const BatchArgs &a, const BatchDesc &d, int lb, BatchLds &L,
                                                    Partial *out) {
    constexpr int NY = (16 * KP + kWave - 1) / kWave;   // doubles of an item's y_i rows per lane
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const BatchBound bd = batch_bound(a.stat[d.set], a.n, d.k, KP);
    const TX *X = static_cast<const TX *>(a.X);
    const int32_t *idx = a.pts + d.pt_off;
    const double *P = a.Pbuf + d.P_off;
    const double *Y = a.Ybuf + d.Y_off;
    const float4 *wt = a.w + d.tile_off * (kTileElems / 4);
    const int64_t nitem = (int64_t)d.ntiles * 4;         // quarter tiles
    if (threadIdx.x == 0) L.run = kKeyNone;
    __syncthreads();
    WaveBest wb{__builtin_huge_val(), __builtin_huge_val(), 0x7fffffff, 0x7fffffff, 0, 0, 0};
    CandList cl{L.cij[wv], L.ckey[wv], 0, a.cap, 0, kKeyNone};
    uint32_t kmin = kKeyNone;
    double *yl = L.y[wv];
    struct ItemLoads {
        float4 w4[4];
        double yr[NY], yj[KP];
        int32_t row0, col;
    };
    auto fetch = [&](int64_t hh, ItemLoads &o) __attribute__((always_inline)) {
        const int64_t t = hh >> 2;
        const int q = (int)(hh & 3);
        const int2 tc = tile_of_index(t, d.nb);
        const float4 *tp = wt + t * (kTileElems / 4) + q * 256 + lane;
#pragma unroll
        for (int g = 0; g < 4; ++g) o.w4[g] = tp[g * 64];
        o.row0 = tc.x * kTile + 16 * q;
        o.col = tc.y * kTile + lane;
        const double *ysrc = Y + (int64_t)o.row0 * KP;
#pragma unroll
        for (int u = 0; u < NY; ++u) {
            const int f = lane + u * kWave;
            o.yr[u] = ysrc[f < 16 * KP ? f : 0];
        }
#pragma unroll
        for (int c = 0; c < KP; ++c) o.yj[c] = Y[(int64_t)o.col * KP + c];
    };
    ItemLoads cur, nxt;
    int64_t h = (int64_t)lb * (kPairBlock / kWave) + wv;
    const int64_t hstep = (int64_t)d.npass * (kPairBlock / kWave);
    if constexpr (PF) {
        if (h < nitem) fetch(h, cur);
        nxt = cur;
    }
    for (; h < nitem; h += hstep) {
        if constexpr (!PF) fetch(h, cur);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < NY; ++u) {
            const int f = lane + u * kWave;
            if (f < 16 * KP) yl[f] = cur.yr[u];
        }
        __builtin_amdgcn_wave_barrier();
        if constexpr (PF)
            if (h + hstep < nitem) fetch(h + hstep, nxt);
        uint32_t key[16];
        uint32_t lmin = kKeyNone;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const double *yi = yl + e * KP;
            double acc = 0.0;
#pragma unroll
            for (int c = 0; c < KP; ++c) {
                const double t2 = yi[c] - cur.yj[c];
                acc = __builtin_fma(t2, t2, acc);
            }
            const float4 &wg = cur.w4[e >> 2];
            const float wv4 = (e & 3) == 0 ? wg.x : (e & 3) == 1 ? wg.y : (e & 3) == 2 ? wg.z : wg.w;
            key[e] = __float_as_uint((float)(acc * (double)wv4));
            lmin = min(lmin, key[e]);
        }
        const uint32_t m = wave_min_u32_fast(lmin);
        kmin = min(kmin, m);
        const uint32_t T2 = item_window(block_run_min(&L.run, m), bd.wa, bd.wb);
        const int32_t row0 = cur.row0, col = cur.col;
        if (m <= T2)
            emit_cands(cl, key, lmin, T2,
                       [=](int e, int32_t &i, int32_t &j) __attribute__((always_inline)) {
                           i = row0 + e;
                           j = col;
                       },
                       wb);
        __builtin_amdgcn_wave_barrier();
        if constexpr (PF) cur = nxt;
    }
    // the window pairs of the block's minimum in FP64 from X, every fourth of
    // the four lists per wavefront (as finish_pass_block)
    if (lane == 0) L.cn[wv] = cl.n;
    __syncthreads();
    const uint32_t run = __builtin_amdgcn_readfirstlane(*(const volatile uint32_t *)&L.run);
    if (run < 0x7f800000u) {
        const uint32_t T2b = item_window(run, bd.wa, bd.wb);
        const int n0 = L.cn[0], n1 = L.cn[1], n2 = L.cn[2], tot = n0 + n1 + n2 + L.cn[3];
        int g = wv;
        uint32_t kv;
        int2 ij;
#pragma unroll 1
        while (next_window_entry(g, tot, n0, n1, n2, L.cij, L.ckey, T2b, kv, ij)) {
            g += kPairBlock / kWave;
            const double r = exact_r_wave<KP, TX>(X, a.ldx, a.n, P, idx[ij.x], idx[ij.y]);
            ++wb.nwin;
            wb.nviol += bound_broken(r, (double)__uint_as_float(kv), bd.e_abs, bd.e_rel);
            lex_pick2(wb.r, wb.i, wb.j, wb.r2, r, ij.x, ij.y, __builtin_huge_val());
        }
    }
    wb.nviol += cl.lost;
    return block_reduce_partial(wb.r, wb.i, wb.j, wb.r2, wb.nwin, wb.nunits, wb.nviol, kmin, cl.limit, out, false,
                                true);
}

template <typename TX>
__global__ __launch_bounds__(kPairBlock, 3) void k_batch_pass(BatchArgs a) {
    __shared__ BatchLds L;
    const int2 bl = a.pass_blk[blockIdx.x];
    const BatchDesc d = a.desc[bl.x];
    Partial *out = a.part + d.part_off + bl.y;
    switch (d.kp) {
        case 2: batch_pass_block<2, false, TX>(a, d, bl.y, L, out); break;
        case 4: batch_pass_block<4, false, TX>(a, d, bl.y, L, out); break;
        case 8: batch_pass_block<8, false, TX>(a, d, bl.y, L, out); break;
        case 12: batch_pass_block<12, false, TX>(a, d, bl.y, L, out); break;
        default: batch_pass_block<16, false, TX>(a, d, bl.y, L, out); break;
    }
}

// Trace entry `it` of problem b from its evaluation f.
__device__ __forceinline__ void batch_record(const BatchArgs &a, const BatchDesc &d, int b, int it, const Partial &f) {
    const BatchBound bd = batch_bound(a.stat[d.set], a.n, d.k, d.kp);
    const bool found = f.r < __builtin_huge_val();
    const uint32_t wkey = f.kmin < 0x7f800000u ? item_window(f.kmin, bd.wa, bd.wb) : 0u;
    const int cert = (found && f.n_viol == 0 && f.limit >= wkey) ? 1 : 0;
    const int64_t tr = (int64_t)b * (a.iters + 1) + it;
    a.tr_min[tr] = f.r;
    if (a.tr_ij) {
        a.tr_ij[2 * tr] = found ? f.i : -1;
        a.tr_ij[2 * tr + 1] = found ? f.j : -1;
    }
    if (a.tr_cert) a.tr_cert[tr] = cert;
}

// Rows [16 s0, 16 s1) of a problem's Y from P in LDS, a slab of 16 per wavefront step.
template <typename TX>
__device__ __forceinline__ void batch_Y(const BatchArgs &a, const BatchDesc &d, const double *sm, int s0, int s1) {
    const double *mu = a.mu + (int64_t)d.set * a.n;
    for (int s = s0 + (int)(threadIdx.x >> 6); s < s1; s += kPairBlock / kWave)
        batch_gemm16<TX>(static_cast<const TX *>(a.X), a.ldx, a.pts + d.pt_off, d.M, a.n, d.k, d.kp, mu, sm,
                         a.Ybuf + d.Y_off, s * 16, a.vx, (a.n & 1) == 0);
}

// Selection, trace entry `it` and (step) update of every problem, then its
// next Y; with sel = 0 only Y, of the starting P.  Block (b, lb) computes the
// rows 64 gt lb .. of problem b's Y; every block of a problem takes the same
// selection and update (identical inputs and arithmetic), block lb = 0 writes
// the trace and P' to the other buffer.  Dynamic LDS: P and the update's two
// vectors, (k + 2) n doubles.
template <typename TX>
__global__ __launch_bounds__(kPairBlock) void k_batch_select(BatchArgs a, int it, int sel, int step) {
    extern __shared__ __align__(16) double sm_batch[];
    const int2 bl = a.sel_blk[blockIdx.x];
    const bool lead = bl.y == 0;
    if (sel && !step && !lead) return;   // the last evaluation: the record alone
    const BatchDesc d = a.desc[bl.x];
    const int n = a.n, k = d.k;
    double *Pn = a.Pnext + d.P_off;
    if (!sel || step) stage_P(a.Pbuf + d.P_off, k * n, sm_batch);
    if (sel) {
        const Partial *part = a.part + d.part_off;
        double best = __builtin_huge_val(), second = __builtin_huge_val();
        int32_t bi = 0x7fffffff, bj = 0x7fffffff, nviol = 0;
        uint32_t kmin = kKeyNone, limit = kKeyNone;
        for (int e = threadIdx.x; e < d.npass; e += kPairBlock) {
            const Partial p = part[e];
            lex_pick2(best, bi, bj, second, p.r, p.i, p.j, p.r2);
            nviol += p.n_viol;
            kmin = min(kmin, p.kmin);
            limit = min(limit, p.limit);
        }
        const Partial f = block_reduce_partial(best, bi, bj, second, 0, 0, nviol, kmin, limit, nullptr, false);
        if (lead && threadIdx.x == 0) batch_record(a, d, bl.x, it, f);
        if (!step) return;
        // (the barrier inside block_reduce_partial has ordered P's staging)
        if (f.r < __builtin_huge_val()) {
            const int32_t *idx = a.pts + d.pt_off;
            batch_update<TX, 1, kMaxK>(static_cast<const TX *>(a.X), a.ldx, n, k, lead ? Pn : nullptr, d.alpha, d.rule,
                                       idx[f.i], idx[f.j], sm_batch);
        } else if (lead) {
            for (int e = threadIdx.x; e < k * n; e += kPairBlock) Pn[e] = sm_batch[e];   // no kept pair: P unchanged
        }
    }
    __syncthreads();
    batch_Y<TX>(a, d, sm_batch, 4 * d.gt * bl.y, min(4 * d.gt * (bl.y + 1), 4 * d.nb));
}

template <int KP> struct KRange;
template <> struct KRange<2> { static constexpr int lo = 1, hi = 2; };
template <> struct KRange<4> { static constexpr int lo = 3, hi = 4; };
template <> struct KRange<8> { static constexpr int lo = 5, hi = 8; };
template <> struct KRange<12> { static constexpr int lo = 9, hi = 12; };
template <> struct KRange<16> { static constexpr int lo = 13, hi = 16; };

// A whole run of problem b in one block (P stays in LDS and, for the
// rescoring, in its first buffer).
template <int KP, bool PF, typename TX>
__device__ __forceinline__ void batch_run_block(BatchArgs &a, const BatchDesc &d, int b, double *sm, BatchLds &L) {
    const int32_t *idx = a.pts + d.pt_off;
    double *P = a.Pbuf + d.P_off;
    stage_P(P, d.k * a.n, sm);
    for (int it = 0; it <= a.iters; ++it) {
        __syncthreads();   // P' (and, before that, the reads of Y) are done
        batch_Y<TX>(a, d, sm, 0, 4 * d.nb);
        __syncthreads();
        const Partial f = batch_pass_block<KP, PF, TX>(a, d, 0, L, nullptr);
        if (threadIdx.x == 0) batch_record(a, d, b, it, f);
        if (!(f.r < __builtin_huge_val())) {
            // a set without a kept pair keeps P: the other entries repeat this one
            if (threadIdx.x == 0)
                for (int r = it + 1; r <= a.iters; ++r) batch_record(a, d, b, r, f);
            return;
        }
        if (it < a.iters)
            batch_update<TX, KRange<KP>::lo, KRange<KP>::hi>(static_cast<const TX *>(a.X), a.ldx, a.n, d.k, P, d.alpha,
                                                             d.rule, idx[f.i], idx[f.j], sm);
    }
}

// Batches of small sets (one_block_per_problem): one block per problem runs all
// its iterations.  PF: sets of more than one tile (an item per wavefront: the
// look ahead would cost it 3%).
template <typename TX, bool PF>
__global__ __launch_bounds__(kPairBlock) void k_batch_run(BatchArgs a) {
    extern __shared__ __align__(16) double sm_batch[];
    __shared__ BatchLds L;
    const BatchProb pr = a.probs[blockIdx.x];
    const BatchDesc d = batch_desc(pr, a.sets[pr.set]);
    switch (d.kp) {
        case 2: batch_run_block<2, PF, TX>(a, d, blockIdx.x, sm_batch, L); break;
        case 4: batch_run_block<4, PF, TX>(a, d, blockIdx.x, sm_batch, L); break;
        case 8: batch_run_block<8, PF, TX>(a, d, blockIdx.x, sm_batch, L); break;
        case 12: batch_run_block<12, PF, TX>(a, d, blockIdx.x, sm_batch, L); break;
        default: batch_run_block<16, PF, TX>(a, d, blockIdx.x, sm_batch, L); break;
    }
}

}  // namespace sap

// ---------------------------------------------------------------- host

using namespace sap;

namespace {

thread_local std::string t_err;

sap_status bfail(sap_status st, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    sap_internal_set_error(buf);
    return st;
}

#define B_HIP(expr)                                                                              \
    do {                                                                                         \
        hipError_t e_ = (expr);                                                                  \
        if (e_ != hipSuccess) {                                                                  \
            (void)hipGetLastError();                                                             \
            return bfail(e_ == hipErrorOutOfMemory ? SAP_ERR_OUT_OF_MEMORY : SAP_ERR_DEVICE,     \
                         "%s: %s", #expr, hipGetErrorString(e_));                                \
        }                                                                                        \
    } while (0)

int kp_of(int k) { return k <= 2 ? 2 : k <= 4 ? 4 : k <= 8 ? 8 : k <= 12 ? 12 : 16; }

int64_t align_up(int64_t v, int64_t a) { return (v + a - 1) / a * a; }

// Host-side plan of one batch call: validated tables and the scratch layout.
struct BatchPlan {
    std::vector<BatchSet> sets;
    std::vector<BatchProb> probs;
    std::vector<int4> tiles;
    std::vector<int32_t> pts;
    std::vector<double> minlen;
    std::vector<BatchDesc> desc;
    bool one_block = false;  // one block per problem and one launch: k_batch_run
    std::vector<int2> pass_blk, sel_blk;
    int64_t ntiles_all = 0, P_total = 0, Y_total = 0, P0_total = 0;
    size_t lds = 0;
    // scratch offsets (bytes); the tables the host fills come first, one copy
    // (the starts' checks lie where Y will: they are read back before it is written)
    size_t o_pts, o_sets, o_probs, o_tiles, o_minlen, o_desc, o_pblk, o_sblk, o_w, o_mu, o_P, o_stat, o_Y, o_part,
        o_P2;
    std::vector<char> tables;   // the tables' host copy
    size_t total = 0;        // bytes of the scratch
    size_t counted = 0;      // with one block per problem: without the block tables, the block results
                             // and the second P.  What scratch_bytes reports and the fixed scratch's
                             // limit counts
};

// Whether one block per problem runs all its iterations (k_batch_run) rather
// than two launches per iteration with more blocks.  The block's iteration
// costs the same for any number of problems up to one per compute unit, and
// grows with the tiles and k; the launches cost 12 us at least, little more
// with the tiles while compute units are idle, and grow with the problems,
// whose blocks repeat the selection.  us per iteration, block and launches:
//   one 64-point block, k <= 12: the block (a call on 30 problems of 40 points,
//     n = 15, 40 iterations 0.84 ms and 1.18 ms; k = 16, n = 64 51.9 and 48.4);
//   two, k <= 4, n <= 128: the block (n = 15, k = 2: 1 problem 9.8 and 13.1,
//     200 10.4 and 16.1, 600 30.4 and 34.8; n = 128, k = 4: 1 problem 18.6 and
//     17.5, 30 18.8 and 18.7; n = 200, k = 5: 30 25.9 and 21.5);
//   more than half a problem per compute unit, up to one: the block for two
//     and k <= 12 (200 problems, n = 15, k = 12 28.2 and 31.8; n = 200, k =
//     16 77 and 74), three and k <= 8 (n = 15, k = 6 25.0 and 27.9; k = 12
//     41.1 and 40.3) and four and k <= 4 (n = 30, k = 4 28.1 and 32.5; k = 6
//     37.1 and 36.5).
bool one_block_per_problem(const BatchPlan &pl, int n, int cus) {
    int nb = 0, k = 0;
    for (const BatchProb &p : pl.probs) {
        nb = std::max(nb, pl.sets[p.set].nb);
        k = std::max(k, p.k);
    }
    const int64_t np = (int64_t)pl.probs.size();
    if ((nb == 1 && k <= 12) || (nb == 2 && k <= 4 && n <= 128)) return true;
    if (np > cus || 2 * np <= cus) return false;
    return (nb == 2 && k <= 12) || (nb == 3 && k <= 8) || (nb == 4 && k <= 4);
}

// Blocks of the two launches.  Pass: one round of resident blocks (three per
// compute unit) dealt to the problems by their quarter tiles, at most one per
// four of them; where every problem gets one block there are as many as
// problems.  Selection: every block repeats its problem's selection and
// update, so there are about as many as compute units (its registers allow one
// block on each), each with whole 64-row groups of Y: the fewest groups that
// take one round (200 problems of five groups: five per block, 200 blocks, and
// not four with 400: 38.5 and 30.7 us per iteration at n = 15, k = 2).
void plan_blocks(BatchPlan &pl, int cus) {
    const int64_t slots = 3 * (int64_t)cus;
    int64_t items = 0, groups = 0, parts = 0;
    for (const BatchProb &p : pl.probs) {
        items += 4ll * pl.sets[p.set].ntiles;
        groups += pl.sets[p.set].nb;
    }
    int32_t gt = (int32_t)std::max<int64_t>(1, (groups + cus - 1) / cus);
    for (int32_t g = gt; g <= 2 * gt; ++g) {
        int64_t blocks = 0;
        for (const BatchProb &p : pl.probs) blocks += (pl.sets[p.set].nb + g - 1) / g;
        if (blocks <= cus) { gt = g; break; }
    }
    pl.desc.resize(pl.probs.size());
    for (size_t b = 0; b < pl.probs.size(); ++b) {
        const BatchProb &p = pl.probs[b];
        const BatchSet &st = pl.sets[p.set];
        BatchDesc &g = pl.desc[b];
        g = batch_desc(p, st);
        g.npass = (int32_t)std::max<int64_t>(1, std::min<int64_t>(st.ntiles, slots * 4 * st.ntiles / items));
        g.gt = gt;
        g.part_off = parts;
        parts += g.npass;
        for (int q = 0; q < g.npass; ++q) pl.pass_blk.push_back(make_int2((int)b, q));
        for (int q = 0; q * gt < st.nb; ++q) pl.sel_blk.push_back(make_int2((int)b, q));
    }
}

// The places of everything in the scratch, and the tables' copy: for one block
// per problem (pl.one_block), or with the block tables, the block results and
// the second P of the two launches.
void plan_layout(BatchPlan &pl, int n) {
    const size_t n_sets = pl.sets.size(), n_problems = pl.probs.size();
    size_t off = 0, extra = 0;
    auto take = [&](size_t bytes) { const size_t o = off; off = (size_t)align_up((int64_t)(off + bytes), 256); return o; };
    auto more = [&](size_t bytes) { const size_t o = off; if (!pl.one_block) { take(bytes); extra += off - o; } return o; };
    pl.o_pts = take(sizeof(int32_t) * pl.pts.size());
    pl.o_sets = take(sizeof(BatchSet) * n_sets);
    pl.o_probs = take(sizeof(BatchProb) * n_problems);
    pl.o_tiles = take(sizeof(int4) * pl.ntiles_all);
    pl.o_minlen = take(sizeof(double) * n_sets);
    pl.o_desc = more(sizeof(BatchDesc) * n_problems);
    pl.o_pblk = more(sizeof(int2) * pl.pass_blk.size());
    pl.o_sblk = more(sizeof(int2) * pl.sel_blk.size());
    pl.tables.resize(off);
    pl.o_w = take(sizeof(float) * (size_t)pl.ntiles_all * kTileElems);
    pl.o_mu = take(sizeof(double) * n_sets * n);
    pl.o_P = take(sizeof(double) * (size_t)pl.P_total);
    pl.o_stat = take(sizeof(BatchStat) * n_sets);
    pl.o_Y = take(sizeof(double) * (size_t)pl.Y_total);
    pl.o_part = more(sizeof(Partial) * pl.pass_blk.size());
    pl.o_P2 = more(sizeof(double) * (size_t)pl.P_total);
    pl.total = off;
    pl.counted = off - extra;
    // (the copy's source: it lives as long as the plan, past the call's last wait)
    auto put = [&](size_t at, const void *p, size_t bytes) { if (bytes) std::memcpy(pl.tables.data() + at, p, bytes); };
    put(pl.o_pts, pl.pts.data(), sizeof(int32_t) * pl.pts.size());
    put(pl.o_sets, pl.sets.data(), sizeof(BatchSet) * n_sets);
    put(pl.o_probs, pl.probs.data(), sizeof(BatchProb) * n_problems);
    put(pl.o_tiles, pl.tiles.data(), sizeof(int4) * pl.tiles.size());
    put(pl.o_minlen, pl.minlen.data(), sizeof(double) * n_sets);
    if (pl.one_block) return;
    put(pl.o_desc, pl.desc.data(), sizeof(BatchDesc) * n_problems);
    put(pl.o_pblk, pl.pass_blk.data(), sizeof(int2) * pl.pass_blk.size());
    put(pl.o_sblk, pl.sel_blk.data(), sizeof(int2) * pl.sel_blk.size());
}

sap_status plan_batch(const void *X, int32_t dtype, int64_t N, int32_t n, int64_t ldx, int32_t n_sets,
                      const int64_t *set_offsets, const int32_t *set_points, const double *set_min_len,
                      int32_t n_problems, const sap_batch_problem *problems, const double *P0, int32_t iters,
                      int32_t cand_cap, double *P_out, double *min_trace, BatchPlan &pl) {
    if (!X || !set_offsets || !set_points || !problems || !P0 || !P_out || !min_trace)
        return bfail(SAP_ERR_INVALID_ARG, "sap_batch_run: null pointer argument");
    if (dtype != SAP_F64 && dtype != SAP_F32) return bfail(SAP_ERR_INVALID_ARG, "dtype must be SAP_F64 or SAP_F32");
    if (N < 2 || N >= (1ll << 31)) return bfail(SAP_ERR_INVALID_ARG, "N must lie in [2, 2^31)");
    if (n < 1) return bfail(SAP_ERR_INVALID_ARG, "n must be >= 1");
    if (ldx < n) return bfail(SAP_ERR_INVALID_ARG, "ldx must be >= n");
    if (n_sets < 1 || n_problems < 1) return bfail(SAP_ERR_INVALID_ARG, "n_sets and n_problems must be >= 1");
    if (n_problems > 65535) return bfail(SAP_ERR_UNSUPPORTED, "at most 65535 problems per call");
    if (iters < 0) return bfail(SAP_ERR_INVALID_ARG, "iters must be >= 0");
    if (cand_cap < 0 || cand_cap > kCandCap) return bfail(SAP_ERR_INVALID_ARG, "cand_cap must lie in [0, %d]", kCandCap);
    if (set_offsets[0] != 0) return bfail(SAP_ERR_INVALID_ARG, "set_offsets[0] must be 0");
    pl.sets.resize(n_sets);
    pl.minlen.resize(n_sets);
    for (int s = 0; s < n_sets; ++s) {
        const int64_t M = set_offsets[s + 1] - set_offsets[s];
        if (M < 2 || M > kBatchMaxPoints)
            return bfail(SAP_ERR_INVALID_ARG, "set %d has %lld points: need 2 .. %d", s, (long long)M, kBatchMaxPoints);
        const double ml = set_min_len ? set_min_len[s] : 0.0;
        if (!(ml >= 0.0) || !std::isfinite(ml)) return bfail(SAP_ERR_INVALID_ARG, "set_min_len[%d] must be finite, >= 0", s);
        pl.minlen[s] = ml;
        BatchSet &b = pl.sets[s];
        b.pt_off = set_offsets[s];
        b.M = (int32_t)M;
        b.nb = (int32_t)((M + kTile - 1) / kTile);
        b.ntiles = b.nb * (b.nb + 1) / 2;
        b.tile_off = pl.ntiles_all;
        b.pad = 0;
        for (int bi = 0; bi < b.nb; ++bi)
            for (int bj = bi; bj < b.nb; ++bj) pl.tiles.push_back(make_int4(bi, bj, s, 0));
        pl.ntiles_all += b.ntiles;
    }
    const int64_t npts = set_offsets[n_sets];
    pl.pts.assign(set_points, set_points + npts);
    for (int64_t e = 0; e < npts; ++e)
        if (pl.pts[e] < 0 || pl.pts[e] >= N)
            return bfail(SAP_ERR_INVALID_ARG, "set_points[%lld] = %d is not a row of X", (long long)e, pl.pts[e]);
    pl.probs.resize(n_problems);
    size_t lds = 0;
    for (int b = 0; b < n_problems; ++b) {
        const sap_batch_problem &q = problems[b];
        if (q.set < 0 || q.set >= n_sets) return bfail(SAP_ERR_INVALID_ARG, "problem %d: set %d out of range", b, q.set);
        if (q.k < 1 || q.k > n) return bfail(SAP_ERR_INVALID_ARG, "problem %d: k = %d outside [1, n]", b, q.k);
        if (q.k > kMaxK) return bfail(SAP_ERR_UNSUPPORTED, "problem %d: k > %d", b, kMaxK);
        if ((int64_t)n * (q.k + 2) > kBatchLdsDoubles)
            return bfail(SAP_ERR_UNSUPPORTED, "problem %d: n (k + 2) must be <= %d", b, kBatchLdsDoubles);
        if (!(q.alpha >= 0.0 && q.alpha <= 1.0)) return bfail(SAP_ERR_INVALID_ARG, "problem %d: alpha outside [0, 1]", b);
        if (q.rule != SAP_STEP_LITERAL && q.rule != SAP_STEP_NORMALIZED)
            return bfail(SAP_ERR_INVALID_ARG, "problem %d: bad rule", b);
        BatchProb &p = pl.probs[b];
        p.set = q.set;
        p.k = q.k;
        p.kp = kp_of(q.k);
        p.rule = q.rule;
        p.alpha = q.alpha;
        p.P_off = pl.P_total;
        p.Y_off = pl.Y_total;
        p.P0_off = pl.P0_total;
        pl.P_total += align_up((int64_t)p.kp * n, 32);
        pl.Y_total += (int64_t)pl.sets[q.set].nb * kTile * p.kp;
        pl.P0_total += (int64_t)n * q.k;
        lds = std::max(lds, sizeof(double) * (size_t)n * (q.k + 2));
    }
    pl.lds = lds;
    int cus = 0, dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) {
        (void)hipGetLastError();
        cus = 256;
    }
    pl.one_block = one_block_per_problem(pl, n, cus);
    if (!pl.one_block) plan_blocks(pl, cus);
    plan_layout(pl, n);
    (void)iters;
    return SAP_OK;
}

// The starts' checks: finite and orthonormal.
sap_status check_P0(const BatchCheck *chk, int n_problems) {
    for (int b = 0; b < n_problems; ++b) {
        if (chk[b].nonfinite) return bfail(SAP_ERR_NONFINITE, "problem %d: P0 holds NaN or Inf", b);
        if (chk[b].err > 1e-6)
            return bfail(SAP_ERR_NOT_ORTHONORMAL, "problem %d: max |P0^T P0 - I| = %.3g > 1e-6", b, chk[b].err);
    }
    return SAP_OK;
}

// Starts that no kernel can read where they lie: copied to the host (an error
// where they are not memory of a device or pinned), checked there in
// k_batch_checkP's order of sums, and put into every P buffer.
sap_status load_starts_by_copy(const BatchPlan &pl, const double *P0, int n, double *Pbuf, double *Pnext,
                               std::vector<BatchCheck> &chk, hipStream_t stream) {
    std::vector<double> h((size_t)pl.P0_total), Pt((size_t)pl.P_total, 0.0);
    B_HIP(hipMemcpyAsync(h.data(), P0, sizeof(double) * h.size(), hipMemcpyDeviceToHost, stream));
    B_HIP(hipStreamSynchronize(stream));
    for (size_t b = 0; b < pl.probs.size(); ++b) {
        const BatchProb &p = pl.probs[b];
        const double *P = h.data() + p.P0_off;
        chk[b] = BatchCheck{0.0, 0, 0};
        for (int e = 0; e < n * p.k; ++e) chk[b].nonfinite |= std::isfinite(P[e]) ? 0 : 1;
        for (int x = 0; x < p.k; ++x)
            for (int y = 0; y < p.k; ++y) {
                double acc = 0.0;
                for (int l = 0; l < n; ++l) acc += P[(size_t)l * p.k + x] * P[(size_t)l * p.k + y];
                chk[b].err = std::max(chk[b].err, std::fabs(acc - (x == y ? 1.0 : 0.0)));   // (a NaN stays out)
            }
        for (int q = 0; q < p.k; ++q)
            for (int l = 0; l < n; ++l) Pt[(size_t)p.P_off + (size_t)q * n + l] = P[(size_t)l * p.k + q];
    }
    B_HIP(hipMemcpyAsync(Pbuf, Pt.data(), sizeof(double) * Pt.size(), hipMemcpyHostToDevice, stream));
    if (Pnext) B_HIP(hipMemcpyAsync(Pnext, Pt.data(), sizeof(double) * Pt.size(), hipMemcpyHostToDevice, stream));
    B_HIP(hipStreamSynchronize(stream));   // (the host vector ends here)
    return SAP_OK;
}

// The events of a timed call, destroyed on every way out.
struct BatchEvents {
    hipEvent_t e[3] = {};
    ~BatchEvents() {
        for (hipEvent_t v : e)
            if (v) (void)hipEventDestroy(v);
    }
};

// Enqueue the whole batch on `stream` with the scratch at `base` (pl.total
// bytes), and wait for it.
sap_status run_batch(const BatchPlan &pl, char *base, const void *X, int32_t dtype, int64_t ldx, int32_t n,
                     int32_t n_sets, int32_t n_problems, const double *P0, int32_t iters, int32_t cand_cap,
                     double *P_out, double *min_trace, int64_t *ij_trace, int32_t *cert_trace, hipStream_t stream,
                     sap_batch_stats *stats, bool timed) {
    BatchArgs a{};
    a.X = X;
    a.ldx = ldx;
    a.n = n;
    const size_t es = dtype == SAP_F64 ? 8 : 4;
    a.vx = (reinterpret_cast<uintptr_t>(X) % 16 == 0) && ((size_t)ldx * es) % 16 == 0;
    a.pts = reinterpret_cast<const int32_t *>(base + pl.o_pts);
    a.sets = reinterpret_cast<const BatchSet *>(base + pl.o_sets);
    a.probs = reinterpret_cast<const BatchProb *>(base + pl.o_probs);
    a.tiles = reinterpret_cast<const int4 *>(base + pl.o_tiles);
    a.w = reinterpret_cast<float4 *>(base + pl.o_w);
    a.mu = reinterpret_cast<double *>(base + pl.o_mu);
    a.stat = reinterpret_cast<BatchStat *>(base + pl.o_stat);
    a.set_min_len = reinterpret_cast<const double *>(base + pl.o_minlen);
    a.desc = reinterpret_cast<const BatchDesc *>(base + pl.o_desc);
    a.chk = reinterpret_cast<BatchCheck *>(base + pl.o_Y);
    a.pass_blk = reinterpret_cast<const int2 *>(base + pl.o_pblk);
    a.sel_blk = reinterpret_cast<const int2 *>(base + pl.o_sblk);
    a.part = reinterpret_cast<Partial *>(base + pl.o_part);
    a.Pbuf = reinterpret_cast<double *>(base + pl.o_P);
    a.Pnext = pl.one_block ? nullptr : reinterpret_cast<double *>(base + pl.o_P2);
    a.Ybuf = reinterpret_cast<double *>(base + pl.o_Y);
    a.P0 = P0;
    a.P_out = P_out;
    a.iters = iters;
    a.cap = cand_cap > 0 ? cand_cap : kCandCap;
    a.tr_min = min_trace;
    a.tr_ij = ij_trace;
    a.tr_cert = cert_trace;
    B_HIP(hipMemcpyAsync(base, pl.tables.data(), pl.tables.size(), hipMemcpyHostToDevice, stream));
    BatchEvents ev;
    if (timed) {
        for (hipEvent_t &v : ev.e) B_HIP(hipEventCreate(&v));
        B_HIP(hipEventRecord(ev.e[0], stream));
    }
    auto launched = [&](const char *what) -> sap_status {
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return bfail(SAP_ERR_DEVICE, "launch of %s: %s", what, hipGetErrorString(e));
        return SAP_OK;
    };
    sap_status st = SAP_OK;
    hipLaunchKernelGGL(k_batch_clear, dim3((n_sets + 255) / 256), dim3(256), 0, stream, a.stat, n_sets);
    if ((st = launched("k_batch_clear")) != SAP_OK) return st;
    int maxM = 0;
    for (const BatchSet &s : pl.sets) maxM = std::max(maxM, s.M);
    const dim3 gm((unsigned)((n + 255) / 256), (unsigned)n_sets), gr((unsigned)((maxM + 3) / 4), (unsigned)n_sets);
    const unsigned gt = (unsigned)std::min<int64_t>(pl.ntiles_all, 8192);
    if (dtype == SAP_F64) {
        hipLaunchKernelGGL(k_batch_mean<double>, gm, dim3(256), 0, stream, a);
        hipLaunchKernelGGL(k_batch_radius<double>, gr, dim3(256), 0, stream, a);
        hipLaunchKernelGGL(k_batch_invd2<double>, dim3(gt), dim3(256), 0, stream, a, pl.ntiles_all);
    } else {
        hipLaunchKernelGGL(k_batch_mean<float>, gm, dim3(256), 0, stream, a);
        hipLaunchKernelGGL(k_batch_radius<float>, gr, dim3(256), 0, stream, a);
        hipLaunchKernelGGL(k_batch_invd2<float>, dim3(gt), dim3(256), 0, stream, a, pl.ntiles_all);
    }
    if ((st = launched("batch precomputation")) != SAP_OK) return st;
    int kpmax = 0;
    for (const BatchProb &p : pl.probs) kpmax = std::max(kpmax, p.kp);
    std::vector<BatchCheck> hc(n_problems);
    int dev = 0;
    hipPointerAttribute_t at{};
    B_HIP(hipGetDevice(&dev));
    const bool in_place = hipPointerGetAttributes(&at, P0) == hipSuccess && kernel_can_read(at, dev);
    if (in_place) {
        hipLaunchKernelGGL(k_batch_loadP, dim3((unsigned)((kpmax * n + 255) / 256), (unsigned)n_problems), dim3(256), 0,
                           stream, a);
        if ((st = launched("k_batch_loadP")) != SAP_OK) return st;
        hipLaunchKernelGGL(k_batch_checkP, dim3((unsigned)n_problems), dim3(256), 0, stream, a);
        if ((st = launched("k_batch_checkP")) != SAP_OK) return st;
    } else {
        (void)hipGetLastError();
        if ((st = load_starts_by_copy(pl, P0, n, a.Pbuf, a.Pnext, hc, stream)) != SAP_OK) return st;
    }
    // inputs checked before the run: orthonormal starts, finite rows, kept pairs
    {
        // (the sets' statistics and the starts' checks lie one behind the other)
        std::vector<char> back(pl.o_Y + sizeof(BatchCheck) * n_problems - pl.o_stat);
        B_HIP(hipMemcpyAsync(back.data(), base + pl.o_stat, back.size(), hipMemcpyDeviceToHost, stream));
        B_HIP(hipStreamSynchronize(stream));
        std::vector<BatchStat> hs(n_sets);
        std::memcpy(hs.data(), back.data(), sizeof(BatchStat) * n_sets);
        if (in_place) std::memcpy(hc.data(), back.data() + (pl.o_Y - pl.o_stat), sizeof(BatchCheck) * n_problems);
        if ((st = check_P0(hc.data(), n_problems)) != SAP_OK) return st;
        int64_t kept = 0;
        for (int s = 0; s < n_sets; ++s) {
            if (hs[s].nonfinite) return bfail(SAP_ERR_NONFINITE, "set %d: X holds NaN or Inf", s);
        }
        for (const BatchProb &p : pl.probs) kept += (int64_t)hs[p.set].kept;
        if (stats) stats->n_pairs = kept;
    }
    if (timed) B_HIP(hipEventRecord(ev.e[1], stream));
    const bool f64 = dtype == SAP_F64, one = pl.one_block;
    int nbmax = 0;
    for (const BatchProb &p : pl.probs) nbmax = std::max(nbmax, pl.sets[p.set].nb);
    auto *const run = nbmax > 1 ? (f64 ? &k_batch_run<double, true> : &k_batch_run<float, true>)
                                : (f64 ? &k_batch_run<double, false> : &k_batch_run<float, false>);
    auto *const sel = f64 ? &k_batch_select<double> : &k_batch_select<float>;
    const void *fn = one ? reinterpret_cast<const void *>(run) : reinterpret_cast<const void *>(sel);
    B_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)pl.lds));
    // Y of the starts, then per iteration the pass and the selection (with the
    // update and the next Y); the last evaluation is only recorded
    const dim3 gp((unsigned)pl.pass_blk.size()), gs((unsigned)pl.sel_blk.size());
    auto select = [&](int it, int evaluated, int step) {
        hipLaunchKernelGGL(sel, gs, dim3(kPairBlock), (uint32_t)pl.lds, stream, a, it, evaluated, step);
        return launched("k_batch_select");
    };
    if (one) {
        hipLaunchKernelGGL(run, dim3((unsigned)n_problems), dim3(kPairBlock), (uint32_t)pl.lds, stream, a);
        if ((st = launched("k_batch_run")) != SAP_OK) return st;
    } else {
        if ((st = select(0, 0, 0)) != SAP_OK) return st;
        for (int it = 0; it <= iters; ++it) {
            if (f64) hipLaunchKernelGGL(k_batch_pass<double>, gp, dim3(kPairBlock), 0, stream, a);
            else hipLaunchKernelGGL(k_batch_pass<float>, gp, dim3(kPairBlock), 0, stream, a);
            if ((st = launched("k_batch_pass")) != SAP_OK) return st;
            if ((st = select(it, 1, it < iters ? 1 : 0)) != SAP_OK) return st;
            if (it < iters) std::swap(a.Pbuf, a.Pnext);
        }
    }
    if (timed) B_HIP(hipEventRecord(ev.e[2], stream));
    hipLaunchKernelGGL(k_batch_storeP, dim3((unsigned)((kpmax * n + 255) / 256), (unsigned)n_problems), dim3(256), 0,
                       stream, a);
    if ((st = launched("k_batch_storeP")) != SAP_OK) return st;
    B_HIP(hipStreamSynchronize(stream));
    if (stats) {
        stats->init_ms = -1.0;
        stats->run_ms = -1.0;
        stats->scratch_bytes = (int64_t)pl.counted;
    }
    if (timed) {
        float t1 = 0.0f, t2 = 0.0f;
        B_HIP(hipEventElapsedTime(&t1, ev.e[0], ev.e[1]));
        B_HIP(hipEventElapsedTime(&t2, ev.e[1], ev.e[2]));
        stats->init_ms = t1;
        stats->run_ms = t2;
    }
    (void)n;
    return SAP_OK;
}

}  // namespace

extern "C" sap_status sap_batch_run(const void *X, int32_t dtype, int64_t N, int32_t n, int64_t ldx, int32_t n_sets,
                                    const int64_t *set_offsets, const int32_t *set_points, const double *set_min_len,
                                    int32_t n_problems, const sap_batch_problem *problems, const double *P0,
                                    int32_t iters, int32_t cand_cap, double *P_out, double *min_trace,
                                    int64_t *ij_trace, int32_t *cert_trace, void *stream, sap_batch_stats *stats) {
    BatchPlan pl;
    sap_status st = plan_batch(X, dtype, N, n, ldx, n_sets, set_offsets, set_points, set_min_len, n_problems, problems,
                               P0, iters, cand_cap, P_out, min_trace, pl);
    if (st != SAP_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(stream);
    void *base = nullptr;
    hipError_t e = hipMalloc(&base, pl.total);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return bfail(e == hipErrorOutOfMemory ? SAP_ERR_OUT_OF_MEMORY : SAP_ERR_DEVICE, "hipMalloc(%zu bytes): %s",
                     pl.total, hipGetErrorString(e));
    }
    st = run_batch(pl, static_cast<char *>(base), X, dtype, ldx, n, n_sets, n_problems, P0, iters, cand_cap, P_out,
                   min_trace, ij_trace, cert_trace, s, stats, stats != nullptr);
    (void)hipStreamSynchronize(s);
    (void)hipFree(base);
    return st;
}

// ---------------------------------------------------------------- allocation-free variant

// The scratch of sap_batch_run_noalloc: a fixed array in device memory.  In
// host code its name only stands for the symbol; its address on a device is
// looked up once per device (hipGetSymbolAddress, with that device current)
// and that address is what the kernels are given.  Each device holds its own
// copy until the process ends; every call on one device shares it.
// The limit counts a batch's data (BatchPlan::counted), which is all that one
// block per problem needs; where what the two launches need beside it does not
// fit, the batch runs that way.
constexpr size_t kStaticScratchBytes = size_t(32) << 20;
static __device__ __align__(256) char scratch[kStaticScratchBytes];

namespace {
std::mutex g_scratch_mu;
std::vector<char *> g_scratch_ptr;   // per device id: the array's device address

sap_status static_scratch(char **out) {
    int dev = 0;
    B_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if ((int)g_scratch_ptr.size() <= dev) g_scratch_ptr.resize((size_t)dev + 1, nullptr);
    if (!g_scratch_ptr[(size_t)dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            (void)hipGetLastError();
            return bfail(SAP_ERR_DEVICE, "hipGetSymbolAddress(scratch) on device %d: %s", dev, hipGetErrorString(e));
        }
        g_scratch_ptr[(size_t)dev] = static_cast<char *>(p);
    }
    *out = g_scratch_ptr[(size_t)dev];
    return SAP_OK;
}
}  // namespace

extern "C" sap_status sap_batch_run_noalloc(const void *X, int32_t dtype, int64_t N, int32_t n, int64_t ldx,
                                            int32_t n_sets, const int64_t *set_offsets, const int32_t *set_points,
                                            const double *set_min_len, int32_t n_problems,
                                            const sap_batch_problem *problems, const double *P0, int32_t iters,
                                            int32_t cand_cap, double *P_out, double *min_trace, int64_t *ij_trace,
                                            int32_t *cert_trace, void *stream, sap_batch_stats *stats) {
    BatchPlan pl;
    sap_status st = plan_batch(X, dtype, N, n, ldx, n_sets, set_offsets, set_points, set_min_len, n_problems, problems,
                               P0, iters, cand_cap, P_out, min_trace, pl);
    if (st != SAP_OK) return st;
    if (pl.counted > kStaticScratchBytes)
        return bfail(SAP_ERR_CAPACITY, "sap_batch_run_noalloc: the batch needs %zu bytes of scratch, above the fixed %zu",
                     pl.counted, kStaticScratchBytes);
    if (pl.total > kStaticScratchBytes) {
        pl.one_block = true;
        plan_layout(pl, n);
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    char *base = nullptr;
    if ((st = static_scratch(&base)) != SAP_OK) return st;
    st = run_batch(pl, base, X, dtype, ldx, n, n_sets, n_problems, P0, iters, cand_cap, P_out, min_trace, ij_trace,
                   cert_trace, s, stats, false);
    (void)hipStreamSynchronize(s);
    return st;
}
