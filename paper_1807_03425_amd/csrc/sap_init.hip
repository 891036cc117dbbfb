// One-time precomputation kernels of a SAP handle (gfx950).
//
//  * column means and the radius max_i ||x_i - mean|| (the error bound of the
//    fused pass is stated in terms of this radius);
//  * plain form: every unit secant s = (x_i - x_j)/||x_i - x_j|| stored once,
//    component-major (n x p), which is the paper's secant matrix S with the
//    secants as columns (Sec. 4);
//  * fused form: 1/d_ij^2 for every pair by direct differences in FP64,
//    packed by 64 x 64 tile, plus the list of short pairs that the coarse
//    FP32 pass cannot resolve and that are therefore evaluated in FP64.
// Pairs that the method drops (duplicates; secants shorter than the length
// threshold of Sec. 7) are masked in both forms.
#include "sap_common.h"
#include "sap_dist.h"

namespace sap {

// ---------------------------------------------------------------- moments

// Block b sums rows [b*rows, (b+1)*rows) of every column, in row order, 16
// rows' loads in flight (one load at a time was a round trip per row).
template <typename TX>
__global__ __launch_bounds__(256) void k_col_partial(const TX *__restrict__ X, int64_t ldx,
                                                     int64_t N, int n, int64_t rows,
                                                     double *__restrict__ part, int32_t *nonfinite) {
    const int64_t r0 = (int64_t)blockIdx.x * rows;
    const int64_t r1 = r0 + rows < N ? r0 + rows : N;
    int bad = 0;
    for (int l = threadIdx.x; l < n; l += blockDim.x) {
        double acc = 0.0;
        int64_t i = r0;
        for (; i + 16 <= r1; i += 16) {
            TX v[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) v[u] = X[(i + u) * ldx + l];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                if (!isfinite(v[u])) bad = 1;
                acc += (double)v[u];
            }
        }
        for (; i < r1; ++i) {
            const double v = (double)X[i * ldx + l];
            if (!isfinite(v)) bad = 1;
            acc += v;
        }
        part[(int64_t)blockIdx.x * n + l] = acc;
    }
    if (bad) atomicOr(nonfinite, 1);
}

__global__ __launch_bounds__(256) void k_col_mean(const double *part, int64_t nblk, int n,
                                                  int64_t N, double *mu) {
    int l = blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= n) return;
    double acc = 0.0;
    int64_t b = 0;
    for (; b + 8 <= nblk; b += 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = part[(b + u) * n + l];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += v[u];
    }
    for (; b < nblk; ++b) acc += part[b * n + l];
    mu[l] = acc / (double)N;
}

// One wavefront per row (grid-stride): ||x_i - mu||, folded into a max on the
// FP64 bits (non-negative doubles order like their bit patterns) -- per block
// first, so that the one address sees an atomic per block and not per row.
template <typename TX>
__global__ __launch_bounds__(256) void k_radius(const TX *__restrict__ X, int64_t ldx,
                                                int64_t N, int n, const double *__restrict__ mu,
                                                unsigned long long *rbits) {
    __shared__ unsigned long long s_max;
    if (threadIdx.x == 0) s_max = 0ull;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    double rmax = 0.0;
    for (int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); row < N; row += (int64_t)gridDim.x * 4) {
        double acc = 0.0;
        for (int l = lane; l < n; l += kWave) {
            const double t = (double)X[row * ldx + l] - mu[l];
            acc += t * t;
        }
        // (a NaN row stays out of the maximum; X is checked for it beforehand)
        rmax = fmax(rmax, sqrt(wave_sum(acc)));
    }
    if (lane == 0) atomicMax(&s_max, (unsigned long long)__double_as_longlong(rmax));
    __syncthreads();
    if (threadIdx.x == 0) atomicMax(rbits, s_max);
}

// ---------------------------------------------------------------- plain form

// S[l * pcols + q] = component l of the unit secant of pair q (computed in
// FP64, stored in T).  Dropped pairs and the padding q >= p hold NaN.
template <typename T>
__global__ __launch_bounds__(256) void k_build_secants(const void *X, int dtype, int64_t ldx,
                                                       int64_t N, int n, double min_len,
                                                       T *S, int64_t pcols, int64_t p,
                                                       unsigned long long *kept,
                                                       unsigned long long *dropped) {
    __shared__ unsigned long long s_kept, s_drop;
    if (threadIdx.x == 0) { s_kept = 0; s_drop = 0; }
    __syncthreads();
    const T nanv = (T)__builtin_nan("");
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < pcols;
         q += (int64_t)gridDim.x * blockDim.x) {
        if (q >= p) {
            for (int l = 0; l < n; ++l) S[(int64_t)l * pcols + q] = nanv;
            continue;
        }
        int64_t i, j;
        decode_pair(q, N, i, j);
        double d2 = 0.0;
        for (int l = 0; l < n; ++l) {
            double t = load_x(X, dtype, i * ldx + l) - load_x(X, dtype, j * ldx + l);
            d2 += t * t;
        }
        double d = sqrt(d2);
        if (d == 0.0 || d < min_len) {
            for (int l = 0; l < n; ++l) S[(int64_t)l * pcols + q] = nanv;
            atomicAdd(&s_drop, 1ull);
            continue;
        }
        for (int l = 0; l < n; ++l) {
            double t = load_x(X, dtype, i * ldx + l) - load_x(X, dtype, j * ldx + l);
            S[(int64_t)l * pcols + q] = (T)(t / d);
        }
        atomicAdd(&s_kept, 1ull);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (s_kept) atomicAdd(kept, s_kept);
        if (s_drop) atomicAdd(dropped, s_drop);
    }
}

template __global__ void k_build_secants<float>(const void *, int, int64_t, int64_t, int,
                                                double, float *, int64_t, int64_t,
                                                unsigned long long *, unsigned long long *);
template __global__ void k_build_secants<double>(const void *, int, int64_t, int64_t, int,
                                                 double, double *, int64_t, int64_t,
                                                 unsigned long long *, unsigned long long *);

// ---------------------------------------------------------------- fused form

// Tile t = (bi, bj), bi <= bj, holds the 64 x 64 pairs
// (i = 64 bi + r, j = 64 bj + c) at float index (r/4)*256 + c*4 + r%4, i.e.
// a lane that owns column c reads rows 4g..4g+3 as one float4 at float4
// index 64 g + c: a wavefront load of 64 consecutive float4 (1 KiB).
//
// ladder[m] = (float)(1 / D_m^2), D_m = D_target * 2^(-m/4), increasing in m.
// A kept pair is counted in bin m when ladder[m] < invd2 <= ladder[m+1]
// (bin 63 takes everything above ladder[63]); the same FP32 comparison later
// decides membership of the close list, so the counts are exact.
//
// One block per tile (grid-stride), distances from tile_dist2; a thread's
// 4 x 4 pairs are twice two consecutive float4 of the tile.  Kept and
// dropped pairs are counted per thread and reduced once per block.
template <typename TX>
__global__ __launch_bounds__(256, 4) void k_build_invd2(const TX *__restrict__ X, int64_t ldx, int64_t N, int n,
                                                        const int2 *__restrict__ tiles, int64_t ntiles,
                                                        double min_len, float4 *__restrict__ invd2,
                                                        const float *__restrict__ ladder, unsigned long long *hist,
                                                        unsigned long long *kept, unsigned long long *dropped,
                                                        uint32_t *__restrict__ tmax) {
    __shared__ __align__(16) DistLds L;
    __shared__ unsigned long long s_hist[64];
    __shared__ unsigned long long s_kept, s_drop;
    __shared__ float s_ladder[64];
    if (threadIdx.x < 64) { s_hist[threadIdx.x] = 0; s_ladder[threadIdx.x] = ladder[threadIdx.x]; }
    if (threadIdx.x == 0) { s_kept = 0; s_drop = 0; }
    const int ty = threadIdx.x >> 4, tx = threadIdx.x & 15;
    const float lad0 = ladder[0];
    unsigned long long nkept = 0, ndrop = 0;
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int2 b = tiles[t];
        __syncthreads();   // the previous tile's rows and chunks have been read
        if (threadIdx.x < 2 * kTile) {
            const int64_t p = (int64_t)(threadIdx.x < kTile ? b.x : b.y) * kTile + (threadIdx.x & (kTile - 1));
            L.row[threadIdx.x] = (int32_t)(p < N ? p : N - 1);
        }
        __syncthreads();
        double d2[4][4];
        tile_dist2(X, ldx, n, L, d2);
        // FULL: a tile of kept and dropped pairs only (off the diagonal, no
        // points past the end), and nothing asked of a length
        auto finish = [&](auto full) __attribute__((always_inline)) {
            constexpr bool FULL = decltype(full)::value;
            const int i0 = b.x * kTile + 4 * ty, j0 = b.y * kTile;
            int drop = 0, kept = 0;
            uint32_t mx = 0u;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int j = j0 + tile_col(tx, q);
                float out[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = i0 + r;
                    const double s = d2[r][q];
                    const bool pair = FULL || (j < N && i < j);
                    const bool keep = pair && s != 0.0 &&
                                      (FULL || !(min_len > 0.0 && tile_shorter(X + i * ldx, X + j * ldx, n, s, min_len)));
                    const float v = keep ? (float)(1.0 / s) : kMaskDropped;
                    mx = max(mx, keep ? __float_as_uint(v) : 0u);
                    drop += pair && !keep;
                    if constexpr (!FULL) kept += keep;
                    if (v > lad0) {
                        int lo = 0;  // largest m with ladder[m] < v
                        for (int hi = 63; lo < hi;) {
                            int mid = (lo + hi + 1) >> 1;
                            if (s_ladder[mid] < v) lo = mid; else hi = mid - 1;
                        }
                        atomicAdd(&s_hist[lo], 1ull);
                    }
                    out[r] = v;
                }
                invd2[t * (kTileElems / 4) + ty * 64 + tile_col(tx, q)] = make_float4(out[0], out[1], out[2], out[3]);
            }
            // the largest of the wavefront's 16 rows (a dropped pair's is negative)
            const uint32_t wmax = wave_max_u32(mx);
            if ((threadIdx.x & (kWave - 1)) == 0) tmax[4 * t + (threadIdx.x >> 6)] = wmax;
            ndrop += drop;
            nkept += FULL ? 16 - drop : kept;
        };
        if (b.x < b.y && ((int64_t)b.y + 1) * kTile <= N && !(min_len > 0.0)) finish(std::true_type{});
        else finish(std::false_type{});
    }
    atomicAdd(&s_kept, nkept);
    atomicAdd(&s_drop, ndrop);
    __syncthreads();
    if (threadIdx.x < 64 && s_hist[threadIdx.x]) atomicAdd(&hist[threadIdx.x], s_hist[threadIdx.x]);
    if (threadIdx.x == 0) {
        if (s_kept) atomicAdd(kept, s_kept);
        if (s_drop) atomicAdd(dropped, s_drop);
    }
}

// Pairs with 1/d^2 above thr become close pairs: masked in the tile array
// and appended (in no particular order; the host sorts the list) to `list`.
// Also folds the largest 1/d^2 left to the coarse pass into *keep_max (as
// float bits: positive floats order like their bit patterns); the coarse
// error bound is stated for the shortest pair the coarse pass still sees.
// One wavefront per four tiles at a time, lanes first over the maxima tmax of
// their quarters (16 rows each): only those above thr are read, a few where
// the short pairs are few.  One atomic per four tiles on the count (they are
// counted first, then read again) and one per block on keep_max: at 12 ns each
// on one address an atomic per pair is what bounds this where the short pairs
// are many.  N = 20000, 222 short pairs: 16 us, 175 with a read of all 800 MB;
// N = 8000, 29940 short pairs: 57 and 444.
__global__ __launch_bounds__(256) void k_mark_close(float4 *invd2, const int2 *tiles,
                                                    int64_t ntiles, const uint32_t *__restrict__ tmax, float thr,
                                                    int2 *list, int64_t cap, unsigned long long *count,
                                                    unsigned *keep_max) {
    __shared__ unsigned s_max;
    if (threadIdx.x == 0) s_max = 0u;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const uint64_t below = (1ull << lane) - 1;
    unsigned mx = 0u;
    for (int64_t q0 = 16 * ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)); q0 < 4 * ntiles;
         q0 += 64 * (int64_t)gridDim.x) {
        const uint32_t tm = lane < 16 && q0 + lane < 4 * ntiles ? tmax[q0 + lane] : 0u;
        const bool over = __uint_as_float(tm) > thr;
        if (!over) mx = max(mx, tm);
        const uint64_t some = __ballot(over);
        if (!some) continue;
        auto quarter = [&](int64_t q, float (&v)[4][4]) __attribute__((always_inline)) {
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const float4 f = invd2[q * (kTileElems / 16) + m * 64 + lane];
                v[m][0] = f.x; v[m][1] = f.y; v[m][2] = f.z; v[m][3] = f.w;
            }
        };
        int hits = 0;   // of the lane
        for (uint64_t todo = some; todo; todo &= todo - 1) {
            float v[4][4];
            quarter(q0 + __ffsll((unsigned long long)todo) - 1, v);
#pragma unroll
            for (int e = 0; e < 16; ++e) hits += v[e / 4][e % 4] > thr;
        }
        for (int o = 1; o < kWave; o <<= 1) hits += __shfl_xor(hits, o, kWave);
        unsigned long long at = 0;
        if (lane == 0) at = atomicAdd(count, (unsigned long long)hits);
        at = __shfl(at, 0, kWave);
        for (uint64_t todo = some; todo; todo &= todo - 1) {
            const int64_t q = q0 + __ffsll((unsigned long long)todo) - 1;
            const int2 b = tiles[q >> 2];
            const int g0 = 4 * (int)(q & 3);
            float v[4][4];
            quarter(q, v);
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                bool hit = false;
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) {
                    const bool one = v[m][rr] > thr;
                    const uint64_t ones = __ballot(one);
                    if (one) {
                        const int64_t to = (int64_t)at + __popcll(ones & below);
                        if (to < cap) list[to] = make_int2(b.x * kTile + 4 * (g0 + m) + rr, b.y * kTile + lane);
                        v[m][rr] = kMaskClose;
                        hit = true;
                    } else if (v[m][rr] > 0.0f) {
                        mx = max(mx, __float_as_uint(v[m][rr]));
                    }
                    at += __popcll(ones);
                }
                if (hit)
                    invd2[q * (kTileElems / 16) + m * 64 + lane] = make_float4(v[m][0], v[m][1], v[m][2], v[m][3]);
            }
        }
    }
    atomicMax(&s_max, mx);
    __syncthreads();
    if (threadIdx.x == 0 && s_max) atomicMax(keep_max, s_max);
}

// P (n x k row-major) -> the FP64 master (k x n), if it is finite and
// max |P^T P - I| <= tol; both verdicts go to host memory.  One block, P in
// chunks of rows through LDS.  The sums of P^T P are shared by up to 32 threads
// per entry (a <= b); where one lies so close to tol that their
// order could decide, they are formed again in the order of the rows, a thread
// per entry, and that is the verdict (a thread per entry throughout took 96 us
// at n = 4800, k = 1).  On the host (P copied out, k^2 serial sums,
// a transposed copy back) a set_P took 39 us at n = 64, k = 6, 54 at n = 1024,
// k = 8 and 30 at n = 4800, k = 1; 20, 27 and 27 with this.
constexpr double kOrthoTol = 1e-6;
constexpr int kLoadP = 1024, kLoadPElems = 4096;
__global__ __launch_bounds__(kLoadP) void k_load_P(const double *__restrict__ P, int n, int k, double tol,
                                                   double *__restrict__ P64t, double *__restrict__ ortho,
                                                   int32_t *__restrict__ finite) {
    __shared__ double s_p[kLoadPElems];
    __shared__ double s_part[kLoadP], s_e[kLoadP / kWave];
    const int tid = threadIdx.x, kk = k * k, chunk = kLoadPElems / k;
    const int part = tid / kk, a = tid % kk / k, b = tid % k;
    int bad = 0;
    // |P^T P - I| of the thread's entry, its rows shared by `parts` threads (0
    // for the threads beside the first of an entry)
    auto deviation = [&](int parts) {
        double acc = 0.0;
        for (int l0 = 0; l0 < n; l0 += chunk) {
            const int rows = n - l0 < chunk ? n - l0 : chunk;
            for (int e = tid; e < rows * k; e += kLoadP) {
                const double v = P[(int64_t)l0 * k + e];
                bad |= !isfinite(v);
                s_p[e] = v;
            }
            __syncthreads();
            if (a <= b && part < parts) {
#pragma unroll 8
                for (int l = part; l < rows; l += parts) acc += s_p[l * k + a] * s_p[l * k + b];
            }
            __syncthreads();
        }
        s_part[tid] = acc;
        __syncthreads();
        if (part > 0 || a > b) return 0.0;
#pragma unroll 8
        for (int q = 1; q < parts; ++q) acc += s_part[q * kk + tid];
        const double d = fabs(acc - (a == b ? 1.0 : 0.0));
        return d >= 0.0 ? d : 0.0;   // (inf - inf off the diagonal: the diagonal is inf)
    };
    double e = deviation(max(1, min(min(kLoadP / kk, 32), n / 8)));
    bad = __syncthreads_or(bad);
    // two orders of a sum of n products are within 2 n 2^-53 sum |p q| of each
    // other, and sum |p q| is below 2 unless a diagonal entry is far above tol
    if (__syncthreads_or(fabs(e - tol) <= (n + 8.0) * 0x1p-50)) e = deviation(1);
    for (int m = 1; m < kWave; m <<= 1) {
        const double o = __shfl_xor(e, m, kWave);
        e = o > e ? o : e;
    }
    if ((tid & (kWave - 1)) == 0) s_e[tid / kWave] = e;
    __syncthreads();
    e = 0.0;
    for (int w = 0; w < kLoadP / kWave; ++w) e = s_e[w] > e ? s_e[w] : e;
    if (tid == 0) {
        *finite = !bad;
        *ortho = e;
    }
    if (bad || e > tol) return;
    for (int x = tid; x < n * k; x += kLoadP) {
        const int q = x / n, l = x % n;
        P64t[x] = P[(int64_t)l * k + q];
    }
}

}  // namespace sap
