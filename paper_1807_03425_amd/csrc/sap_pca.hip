// Algorithm 1's initial projection (Sec. 4, Algorithm 1 step 2): the first k
// columns of U in the SVD S = U Sigma V^T of the secant matrix S (every kept
// unit secant as a column), i.e. the top-k eigenvectors of
//     C = S S^T = sum_{kept i<j} s_ij s_ij^T,   sigma_c^2 = its eigenvalues,
// computed without forming S (gfx950, FP64 throughout):
//   k_pca_w     w_ij = 1/d_ij^2 for every kept pair (0 for dropped pairs,
//               i >= j and padding), by direct differences, 64 x 64 tiles;
//   k_pca_z     z_i = sum_j w_ij (x_i - x_j): the differences are formed
//               directly, never as deg_i x_i - (W X)_i, whose two terms cancel
//               on close pairs;
//   k_pca_gram  C = sum_i (x_i - mean) z_i^T (exact: sum_i z_i = 0, and
//               1/2 sum_ij w_ij (x_i - x_j)(x_i - x_j)^T = sum_i x_i z_i^T),
//               symmetrised;
//   subspace iteration on C with a block of b >= k vectors: a Chebyshev
//   filter of the unwanted part of the spectrum (products C V: k_pca_mv),
//   orthonormalisation (k_pca_orth), and a Rayleigh-Ritz step (k_pca_rr:
//   V^T C V diagonalised by a parallel cyclic Jacobi) that reports the Ritz
//   values and the residuals of the first k Ritz vectors.
#include "sap_common.h"
#include "sap_dist.h"

namespace sap {

constexpr int kPcaMaxB = 32;   // subspace block size

// 1/d^2 of every kept pair of tile t = (bi, bj), row-major 64 x 64 FP64
// (distances from tile_dist2); zero for dropped pairs (duplicates, d <
// min_len), i >= j and padding.
template <typename TX>
__global__ __launch_bounds__(256, 4) void k_pca_w(const TX *__restrict__ X, int64_t ldx, int64_t N, int n,
                                                  const int2 *__restrict__ tiles, int64_t ntiles, double min_len,
                                                  double *__restrict__ W) {
    __shared__ __align__(16) DistLds L;
    const int ty = threadIdx.x >> 4, tx = threadIdx.x & 15;
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
        const int64_t i0 = (int64_t)b.x * kTile + 4 * ty, j0 = (int64_t)b.y * kTile;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            double v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const double s = d2[r][q];
                const int64_t ii = i0 + r, jj = j0 + tile_col(tx, q);
                const bool kept = jj < N && ii < jj && s != 0.0 &&
                                  !(min_len > 0.0 && tile_shorter(X + ii * ldx, X + jj * ldx, n, s, min_len));
                v[q] = kept ? 1.0 / s : 0.0;
            }
            double2 *o = reinterpret_cast<double2 *>(W + t * kTileElems + (4 * ty + r) * kTile + 2 * tx);
            o[0] = make_double2(v[0], v[1]);
            o[16] = make_double2(v[2], v[3]);
        }
    }
}

// z_i = sum_j w_ij (x_i - x_j) for the 64 rows of point block I, 64 components
// and a range of column blocks J (one of S), into partial sp of Z (Zp: S x N
// x n).  Thread (ty, tx) keeps z of rows 4 ty .. and components 4 tx .. with
// its x_i in registers; 32 columns at a time of the w tile (transposed when
// J > I) and of X_J are staged in LDS, where 4 reads of 16 bytes feed 32
// FP64 instructions.  Bound by FP64 VALU issue (2 per row, column and
// component).  S fills the chip when there are few point blocks: N = 4000, n
// = 64 has 63, and one block each walking all J took 1633 us, against 143 us
// with 16 ranges.  The component chunks of one (I, range) sit at the same
// place of eight consecutive groups of blocks, i.e. on one die, and share its
// cached w tiles.
constexpr int kPcaJ = 32;
template <typename TX>
__global__ __launch_bounds__(256, 3) void k_pca_z(const TX *__restrict__ X, int64_t ldx, int64_t N, int n, int64_t nb,
                                                  int nch, int S, const double *__restrict__ W,
                                                  double *__restrict__ Zp) {
    __shared__ __align__(16) double s_w[kPcaJ][kTile + 2];
    __shared__ __align__(16) double s_x[kPcaJ][kTile + 2];
    const int64_t slot = blockIdx.x >> 3;
    const int ch = (int)(slot % nch);
    const int64_t g = (slot / nch) * 8 + (blockIdx.x & 7);
    if (g >= nb * S) return;
    const int64_t I = g % nb;
    const int sp = (int)(g / nb);
    const int64_t J0 = nb * sp / S, J1 = nb * (sp + 1) / S;
    const int l0 = ch * kTile;
    const int ty = threadIdx.x >> 4, tx = threadIdx.x & 15;
    double xi[4][4], z[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t i = I * kTile + 4 * ty + r;
            const int l = l0 + 4 * tx + q;
            xi[r][q] = (double)X[(i < N ? i : N - 1) * ldx + (l < n ? l : n - 1)];
            z[r][q] = 0.0;
        }
#pragma unroll 1
    for (int64_t J = J0; J < J1; ++J) {
        const int64_t bi = I < J ? I : J, bj = I < J ? J : I;
        const double *T = W + (bi * nb - bi * (bi - 1) / 2 + (bj - bi)) * kTileElems;
#pragma unroll 1
        for (int j0 = 0; j0 < kTile; j0 += kPcaJ) {
            __syncthreads();   // the previous columns have been read
#pragma unroll
            for (int u = 0; u < kPcaJ * kTile / 256; ++u) {
                const int e = threadIdx.x + u * 256;
                if (I < J) {                       // tile rows are i: read along j, store transposed
                    const int jj = e % kPcaJ, ii = e / kPcaJ;
                    s_w[jj][ii] = T[ii * kTile + j0 + jj];
                } else {                           // tile rows are j
                    const int ii = e % kTile, jj = e / kTile, j = j0 + jj;
                    // (the diagonal tile holds i < j only)
                    s_w[jj][ii] = I > J || j < ii ? T[j * kTile + ii] : j > ii ? T[ii * kTile + j] : 0.0;
                }
                const int cc = e % kTile, jr = e / kTile;
                const int64_t j = J * kTile + j0 + jr;
                s_x[jr][cc] = (double)X[(j < N ? j : N - 1) * ldx + (l0 + cc < n ? l0 + cc : n - 1)];
            }
            __syncthreads();
#pragma unroll 4
            for (int jj = 0; jj < kPcaJ; ++jj) {
                const double2 *pw = reinterpret_cast<const double2 *>(&s_w[jj][4 * ty]);
                const double2 *px = reinterpret_cast<const double2 *>(&s_x[jj][4 * tx]);
                const double2 w0 = pw[0], w1 = pw[1], x0 = px[0], x1 = px[1];
                const double w[4] = {w0.x, w0.y, w1.x, w1.y}, x[4] = {x0.x, x0.y, x1.x, x1.y};
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int q = 0; q < 4; ++q) z[r][q] = __builtin_fma(w[r], xi[r][q] - x[q], z[r][q]);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t i = I * kTile + 4 * ty + r;
        if (i < N) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int l = l0 + 4 * tx + q;
                if (l < n) Zp[((int64_t)sp * N + i) * n + l] = z[r][q];
            }
        }
    }
}

// Z <- sum of its S partials, into the first.
__global__ __launch_bounds__(256) void k_pca_zsum(double *__restrict__ Zp, int64_t nz, int S) {
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < nz; e += (int64_t)gridDim.x * 256) {
        double acc = Zp[e];
        for (int s = 1; s < S; ++s) acc += Zp[(int64_t)s * nz + e];
        Zp[e] = acc;
    }
}

// Partial r of C[a][b] = sum_i (x_ia - mu_a) z_ib (row-major n x n,
// unsymmetrised): the rows i of R ranges (blockIdx.y), the 64 x 64 tile
// blockIdx.x of C, 4 x 4 entries per thread.  The ranges fill the chip: one
// block per tile took 1621 us at N = 4000, n = 64 (one tile), against 10 us.
template <typename TX>
__global__ __launch_bounds__(256) void k_pca_gram(const TX *__restrict__ X, int64_t ldx, int64_t N, int n,
                                                  const double *__restrict__ mu, const double *__restrict__ Z,
                                                  double *__restrict__ Cp) {
    __shared__ __align__(16) double s_x[kPcaJ][kTile + 2];
    __shared__ __align__(16) double s_z[kPcaJ][kTile + 2];
    const int gn = (n + kTile - 1) / kTile;
    const int a0 = (int)(blockIdx.x / gn) * kTile, b0 = (int)(blockIdx.x % gn) * kTile;
    const int64_t i0 = N * blockIdx.y / gridDim.y, i1 = N * (blockIdx.y + 1) / gridDim.y;
    const int ty = threadIdx.x >> 4, tx = threadIdx.x & 15;
    double acc[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[r][q] = 0.0;
    for (int64_t ib = i0; ib < i1; ib += kPcaJ) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kPcaJ * kTile / 256; ++u) {
            const int e = threadIdx.x + u * 256;
            const int cc = e % kTile, rr = e / kTile;
            const int64_t i = ib + rr < i1 ? ib + rr : i1 - 1;
            const int la = a0 + cc < n ? a0 + cc : n - 1, lb = b0 + cc < n ? b0 + cc : n - 1;
            const double xv = (double)X[i * ldx + la] - mu[la], zv = Z[i * n + lb];
            s_x[rr][cc] = ib + rr < i1 ? xv : 0.0;
            s_z[rr][cc] = ib + rr < i1 ? zv : 0.0;
        }
        __syncthreads();
#pragma unroll 4
        for (int rr = 0; rr < kPcaJ; ++rr) {
            const double2 *pa = reinterpret_cast<const double2 *>(&s_x[rr][4 * ty]);
            const double2 *pb = reinterpret_cast<const double2 *>(&s_z[rr][4 * tx]);
            const double2 x0 = pa[0], x1 = pa[1], z0 = pb[0], z1 = pb[1];
            const double x[4] = {x0.x, x0.y, x1.x, x1.y}, z[4] = {z0.x, z0.y, z1.x, z1.y};
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[r][q] = __builtin_fma(x[r], z[q], acc[r][q]);
        }
    }
    double *out = Cp + (int64_t)blockIdx.y * n * n;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int a = a0 + 4 * ty + r, b = b0 + 4 * tx + q;
            if (a < n && b < n) out[(int64_t)a * n + b] = acc[r][q];
        }
}

// Cs <- (C + C^T) / 2 from the R partials of C, rows and columns padded with
// zeros to ld (a multiple of 64: the products below need no edge).
__global__ __launch_bounds__(256) void k_pca_sym(const double *__restrict__ Cp, int R, int n, int ld,
                                                 double *__restrict__ Cs) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)ld * ld) return;
    const int a = (int)(e / ld), b = (int)(e % ld);
    double s1 = 0.0, s2 = 0.0;
    if (a < n && b < n) {
        const double *c1 = Cp + (int64_t)a * n + b, *c2 = Cp + (int64_t)b * n + a;
        const int64_t nn = (int64_t)n * n;
        int r = 0;
        for (; r + 8 <= R; r += 8) {   // (sixteen loads in flight; the sums in order)
            double u[8], v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) { u[q] = c1[(r + q) * nn]; v[q] = c2[(r + q) * nn]; }
#pragma unroll
            for (int q = 0; q < 8; ++q) { s1 += u[q]; s2 += v[q]; }
        }
        for (; r < R; ++r) { s1 += c1[r * nn]; s2 += c2[r * nn]; }
    }
    Cs[e] = 0.5 * (s1 + s2);
}

// ---------------------------------------------------------------- subspace iteration
//
// A block of vectors is stored component-contiguous: kPcaMaxB columns of ld
// doubles, the components past n and the columns past b zero.

// Deterministic start block, entries in [-1, 1) from a counter hash
// (splitmix64 of the element index).
__device__ __forceinline__ double pca_hash(uint64_t x) {
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    x ^= x >> 31;
    return (double)(x >> 11) * (2.0 / 9007199254740992.0) - 1.0;
}

__global__ void k_pca_start(double *__restrict__ V, int n, int b, int ld, int ne) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= ne) return;
    const int c = e / ld, l = e % ld;
    V[e] = c < b && l < n ? pca_hash((uint64_t)l * b + c) : 0.0;
}

// 4 consecutive components of a column (16-byte aligned).
__device__ __forceinline__ void pca_load4(const double *__restrict__ p, double (&o)[4]) {
    const double2 a = reinterpret_cast<const double2 *>(p)[0], b = reinterpret_cast<const double2 *>(p)[1];
    o[0] = a.x; o[1] = a.y; o[2] = b.x; o[3] = b.y;
}

// Out = alpha C In + beta In + gamma Prev, one block per 16 rows: v_mfma_f64_16x16x4f64 with the contraction
// over 16-component slices dealt to the four wavefronts (lane (m, kk) holds
// components 4 kk .. of row / column m), their sums added in order in LDS.
// One thread per output element walking C's row took 17.8 us at n = 64.
template <int BT>
__global__ __launch_bounds__(256) void k_pca_mv(const double *__restrict__ Cs, int ld, const double *__restrict__ In,
                                                const double *__restrict__ Prev, double alpha, double beta,
                                                double gamma, double *__restrict__ Out) {
    __shared__ double s_p[4][BT][4][kWave];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int m = lane & 15, kk = lane >> 4;
    const int row0 = blockIdx.x * 16;
    const double *cr = Cs + (int64_t)(row0 + m) * ld + 4 * kk;
    const double *vc = In + (int64_t)m * ld + 4 * kk;
    double4_t acc[BT];
#pragma unroll
    for (int t = 0; t < BT; ++t) acc[t] = double4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int l0 = 16 * w; l0 < ld; l0 += 64) {
        double a[4], v[BT][4];
        pca_load4(cr + l0, a);
#pragma unroll
        for (int t = 0; t < BT; ++t) pca_load4(vc + (int64_t)16 * t * ld + l0, v[t]);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int t = 0; t < BT; ++t)
                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], v[t][u], acc[t], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < BT; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u) s_p[w][t][u][lane] = acc[t][u];
    __syncthreads();
    // element u of a lane: row kk + 4 u, column m of the tile
    const int u = threadIdx.x >> 6;
#pragma unroll
    for (int t = 0; t < BT; ++t) {
        const double s = (s_p[0][t][u][lane] + s_p[1][t][u][lane]) + (s_p[2][t][u][lane] + s_p[3][t][u][lane]);
        const int64_t e = (int64_t)(16 * t + m) * ld + row0 + kk + 4 * u;
        double o = alpha * s;
        if (beta != 0.0) o = __builtin_fma(beta, In[e], o);
        if (gamma != 0.0) o = __builtin_fma(gamma, Prev[e], o);
        Out[e] = o;
    }
}

// Out = alpha A + beta B, element by element.
__global__ __launch_bounds__(256) void k_pca_lin(const double *__restrict__ A, const double *__restrict__ B,
                                                 double alpha, double beta, int ne, double *__restrict__ Out) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e < ne) Out[e] = __builtin_fma(beta, B[e], alpha * A[e]);
}

// A round's whole Chebyshev filter in one block, for n <= LD: the first term
// Y = f1 W + f0 V, then deg - 1 times (X, Y) <- (Y, a_d C Y + b_d Y + g_d X).  A
// wavefront owns a 16 x 16 tile of the terms; its rows of C stay in registers
// as MFMA operands, its own elements of X and Y too, and Y goes around through
// two buffers in LDS (rows of LD + 2: the 16 columns of a read cover every
// bank).  Products and sums in k_pca_mv's order.  Bound by the MFMA issue, LD /
// 4 of 64 cycles per step: 1.0 us a step at n = 64 and 16 columns, where a
// launch of k_pca_mv per step took 3.5.
struct PcaCoef {
    double a[32], b[32], g[32];   // of term d, d = 2 .. deg <= 32, at d - 1
};
template <int BT, int LD>
__global__ __launch_bounds__(LD / 16 * BT * kWave) void k_pca_cheb(const double *__restrict__ Cs,
                                                                  const double *__restrict__ V,
                                                                  const double *__restrict__ W, double f1, double f0,
                                                                  int deg, PcaCoef co, double *__restrict__ Out) {
    __shared__ __align__(16) double s_y[2][16 * BT][LD + 2];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int m = lane & 15, kk = lane >> 4;
    const int row0 = 16 * (w % (LD / 16)), col = 16 * (w / (LD / 16)) + m;
    double c[LD / 16][4];
#pragma unroll
    for (int q = 0; q < LD / 16; ++q) pca_load4(Cs + (int64_t)(row0 + m) * LD + 16 * q + 4 * kk, c[q]);
    // element u of a lane: row row0 + kk + 4 u, column col
    double x[4], y[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = col * LD + row0 + kk + 4 * u;
        x[u] = V[e];
        y[u] = __builtin_fma(f0, x[u], f1 * W[e]);
        s_y[0][col][row0 + kk + 4 * u] = y[u];
    }
    __syncthreads();
    const int c0 = col - m;
    for (int d = 1; d < deg; ++d) {
        const double *v0 = &s_y[(d - 1) & 1][c0 + m][4 * kk];
        double4_t acc[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = double4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < LD / 16; ++q) {
            double v[4];
            pca_load4(v0 + 16 * q, v);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                acc[q & 3] = __builtin_amdgcn_mfma_f64_16x16x4f64(c[q][u], v[u], acc[q & 3], 0, 0, 0);
        }
        const double al = co.a[d], be = co.b[d], ga = co.g[d];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            double o = al * ((acc[0][u] + acc[1][u]) + (acc[2][u] + acc[3][u]));
            if (be != 0.0) o = __builtin_fma(be, y[u], o);
            if (ga != 0.0) o = __builtin_fma(ga, x[u], o);
            x[u] = y[u];
            y[u] = o;
            s_y[d & 1][col][row0 + kk + 4 * u] = o;
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) Out[col * LD + row0 + kk + 4 * u] = y[u];
}

constexpr int kPcaBlock = 1024;                  // threads of the one-block kernels
constexpr int kPcaWaves = kPcaBlock / kWave;

struct PcaLds {
    double g[kPcaMaxB][kPcaMaxB + 1];            // Gram / projected matrix
    double part[kPcaWaves][2][4][kWave];         // wavefronts' partial products
};

// L.g[a][c] = sum_l A[a][l] B[c][l] for the BT x BT tiles of 16 columns each
// (only the tiles on and above the diagonal when sym), all threads.
template <int BT>
__device__ __forceinline__ void pca_gram_block(const double *A, const double *B, int ld, PcaLds &L) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int m = lane & 15, kk = lane >> 4;
#pragma unroll 1
    for (int ta = 0; ta < BT; ++ta) {
        double4_t acc[BT];
#pragma unroll
        for (int t = 0; t < BT; ++t) acc[t] = double4_t{0.0, 0.0, 0.0, 0.0};
        for (int l0 = 16 * w; l0 < ld; l0 += 16 * kPcaWaves) {
            double a[4], v[BT][4];
            pca_load4(A + (int64_t)(16 * ta + m) * ld + l0 + 4 * kk, a);
#pragma unroll
            for (int t = 0; t < BT; ++t) pca_load4(B + (int64_t)(16 * t + m) * ld + l0 + 4 * kk, v[t]);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int t = 0; t < BT; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], v[t][u], acc[t], 0, 0, 0);
        }
        __syncthreads();   // the previous tile row's partials have been read
#pragma unroll
        for (int t = 0; t < BT; ++t)
#pragma unroll
            for (int u = 0; u < 4; ++u) L.part[w][t][u][lane] = acc[t][u];
        __syncthreads();
        for (int e = threadIdx.x; e < BT * 256; e += kPcaBlock) {
            const int t = e >> 8, u = (e >> 6) & 3, ln = e & 63;
            double s = 0.0;
            for (int q = 0; q < kPcaWaves; ++q) s += L.part[q][t][u][ln];
            L.g[16 * ta + (ln >> 4) + 4 * u][16 * t + (ln & 15)] = s;
        }
    }
    __syncthreads();
}

// Sum of x over the block's wavefronts' lanes, in every thread (fixed order).
__device__ __forceinline__ double pca_block_sum(double x, double *sb) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, kWave);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sb[threadIdx.x >> 6] = x;
    __syncthreads();
    double t = 0.0;
    for (int w = 0; w < kPcaWaves; ++w) t += sb[w];
    return t;
}

// The general orthonormalisation of the b columns in place: classical
// Gram-Schmidt, twice per column; a column that cancels to below 1e-10 of
// its norm is replaced by a hashed vector and orthogonalised again.
__device__ void pca_cgs2(double *V, int n, int b, int ld, int seed, double *sb) {
    for (int c = 0; c < b; ++c) {
        double *vc = V + (int64_t)c * ld;
        for (int attempt = 0; attempt < 2; ++attempt) {
            double s = 0.0;
            for (int l = threadIdx.x; l < n; l += kPcaBlock) s = __builtin_fma(vc[l], vc[l], s);
            const double nrm0 = sqrt(pca_block_sum(s, sb));
            for (int pass = 0; pass < 2; ++pass) {
                double d[kPcaMaxB];
                for (int a = 0; a < c; ++a) {
                    double t = 0.0;
                    for (int l = threadIdx.x; l < n; l += kPcaBlock) t = __builtin_fma(V[(int64_t)a * ld + l], vc[l], t);
                    d[a] = pca_block_sum(t, sb);
                }
                for (int l = threadIdx.x; l < n; l += kPcaBlock) {
                    double x = vc[l];
                    for (int a = 0; a < c; ++a) x -= d[a] * V[(int64_t)a * ld + l];
                    vc[l] = x;
                }
                __syncthreads();
            }
            s = 0.0;
            for (int l = threadIdx.x; l < n; l += kPcaBlock) s = __builtin_fma(vc[l], vc[l], s);
            const double nrm = sqrt(pca_block_sum(s, sb));
            if (nrm > 1e-10 * nrm0 && nrm > 1e-300) {
                for (int l = threadIdx.x; l < n; l += kPcaBlock) vc[l] = vc[l] / nrm;
                __syncthreads();
                break;
            }
            // lost to cancellation: a fresh direction (the loop orthogonalises it)
            for (int l = threadIdx.x; l < n; l += kPcaBlock)
                vc[l] = pca_hash(0x51A9ull + (uint64_t)seed * 7919ull + (uint64_t)(c * n + l) * 131ull);
            __syncthreads();
        }
    }
}

// Orthonormalise the b columns of V in place (one block): Cholesky of the Gram
// matrix and forward substitution, twice (the second pass brings the first's
// cond^2 u64 down to u64).  A column whose pivot falls below 1e-12 of its
// squared norm (so that the first pass would lose more than six digits) sends
// the block to pca_cgs2, which replaces what is linearly dependent.  Column by
// column Gram-Schmidt on everything took 140 us at n = 64, b = 14, a block
// reduction per inner product; this takes 19 us.
template <int BT>
__global__ __launch_bounds__(kPcaBlock) void k_pca_orth(double *__restrict__ V, int n, int b, int ld, int seed) {
    constexpr int B = 16 * BT;
    __shared__ PcaLds L;
    __shared__ double col[2][kPcaMaxB];
    __shared__ double sb[kPcaWaves];
    const int i = threadIdx.x / kPcaMaxB, m = threadIdx.x % kPcaMaxB;   // element of the Gram matrix
#pragma unroll 1
    for (int pass = 0; pass < 2; ++pass) {
        pca_gram_block<BT>(V, V, ld, L);
        // Cholesky, element (i, m) of the lower triangle in its thread; the
        // padding columns are those of the identity
        const bool in = i < b && m <= i;
        double g = in ? L.g[i][m] : 0.0;
        const double diag = m < b ? L.g[m][m] : 1.0;   // column m's squared norm
        bool ok = true;
        __syncthreads();
        for (int j = 0; j < b; ++j) {
            if (m == j && in) col[j & 1][i] = g;
            __syncthreads();
            const double piv = col[j & 1][j];
            // every thread sees every pivot; column j's norm is in the threads m = j
            if (m == j && !(piv > 1e-12 * diag && piv > 1e-300)) ok = false;
            if (in && m == j) L.g[i][j] = i == j ? 1.0 / sqrt(piv) : g / sqrt(piv);
            if (in && m > j) g -= col[j & 1][i] * col[j & 1][m] / piv;
        }
        if (__syncthreads_or(ok ? 0 : 1)) {
            pca_cgs2(V, n, b, ld, seed, sb);
            return;
        }
        // v_j <- (v_j - sum_{m < j} L[j][m] q_m) / L[j][j], a row of V per thread
        for (int l = threadIdx.x; l < n; l += kPcaBlock) {
            double v[B];
#pragma unroll
            for (int j = 0; j < B; ++j) v[j] = j < b ? V[(int64_t)j * ld + l] : 0.0;
#pragma unroll
            for (int j = 0; j < B; ++j) {
                if (j < b) {
#pragma unroll
                    for (int q = 0; q < j; ++q) {
                        if (q % 8 == 0) asm volatile("" ::: "memory");   // (no more of L in registers at once)
                        v[j] = __builtin_fma(-L.g[j][q], v[q], v[j]);
                    }
                    v[j] *= L.g[j][j];
                }
            }
#pragma unroll
            for (int j = 0; j < B; ++j)
                if (j < b) V[(int64_t)j * ld + l] = v[j];
        }
        __syncthreads();
    }
}

// Rayleigh-Ritz on the orthonormal V with W = C V: H = (V^T W + W^T V) / 2
// (b x b), diagonalised by a parallel cyclic Jacobi (round-robin pairs, b/2
// rotations per step), Ritz values sorted descending, V2 = V Q, W2 = W Q,
// and out[0..b) = Ritz values, out[b] = max_{c<k} ||W2_c - theta_c V2_c|| /
// theta_0.  One block.
template <int BT>
__global__ __launch_bounds__(kPcaBlock) void k_pca_rr(const double *__restrict__ V, const double *__restrict__ W,
                                                      double *__restrict__ V2, double *__restrict__ W2, int n, int b,
                                                      int k, int ld, double *__restrict__ out) {
    __shared__ PcaLds L;
    __shared__ double Q[kPcaMaxB][kPcaMaxB + 1];
    __shared__ double rot[kPcaMaxB / 2][2];
    __shared__ int rpq[kPcaMaxB / 2][2];
    __shared__ int perm[kPcaMaxB];
    __shared__ double theta[kPcaMaxB];
    __shared__ double sb[kPcaWaves], res[kPcaWaves];
    auto &A = L.g;
    const int bp = b + (b & 1);   // even number of players; the pad has A = 0
    const int ea = threadIdx.x / kPcaMaxB, ec = threadIdx.x % kPcaMaxB;
    pca_gram_block<BT>(V, W, ld, L);
    {
        const double h = ea < b && ec < b ? 0.5 * (A[ea][ec] + A[ec][ea]) : 0.0;
        __syncthreads();
        A[ea][ec] = h;
        Q[ea][ec] = ea == ec ? 1.0 : 0.0;
    }
    __syncthreads();
    for (int sweep = 0; sweep < 30; ++sweep) {
        const double av = ea < bp && ec < bp ? A[ea][ec] * A[ea][ec] : 0.0;
        const double off = pca_block_sum(ea < ec ? av : 0.0, sb), dia = pca_block_sum(ea == ec ? av : 0.0, sb);
        if (off <= 1e-32 * dia) break;   // the same in every thread
        for (int step = 0; step < bp - 1; ++step) {
            if (threadIdx.x < bp / 2) {
                const int m = threadIdx.x;
                const int pa = m == 0 ? 0 : ((m - 1 + step) % (bp - 1)) + 1;
                const int mq = bp - 1 - m;
                const int pb = ((mq - 1 + step) % (bp - 1)) + 1;
                const int p = min(pa, pb), q = max(pa, pb);
                const double apq = A[p][q];
                double c = 1.0, s = 0.0;
                if (apq != 0.0) {
                    const double tau = (A[q][q] - A[p][p]) / (2.0 * apq);
                    const double t = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
                    c = 1.0 / sqrt(1.0 + t * t);
                    s = t * c;
                }
                rot[m][0] = c; rot[m][1] = s;
                rpq[m][0] = p; rpq[m][1] = q;
            }
            __syncthreads();
            // rows p, q of A  (A <- J^T A); at most 16 x 32 elements
            const int m = threadIdx.x / bp, j = threadIdx.x % bp;
            const bool on = m < bp / 2;
            const int p = on ? rpq[m][0] : 0, q = on ? rpq[m][1] : 0;
            const double c = on ? rot[m][0] : 1.0, s = on ? rot[m][1] : 0.0;
            if (on) {
                const double ap = A[p][j], aq = A[q][j];
                A[p][j] = c * ap - s * aq;
                A[q][j] = s * ap + c * aq;
            }
            __syncthreads();
            // columns p, q of A and of Q  (A <- A J, Q <- Q J)
            if (on) {
                const double ap = A[j][p], aq = A[j][q];
                A[j][p] = c * ap - s * aq;
                A[j][q] = s * ap + c * aq;
                const double qp = Q[j][p], qq = Q[j][q];
                Q[j][p] = c * qp - s * qq;
                Q[j][q] = s * qp + c * qq;
            }
            __syncthreads();
        }
    }
    if (threadIdx.x < kPcaMaxB) perm[threadIdx.x] = threadIdx.x;
    __syncthreads();
    if (threadIdx.x < b) {
        // descending order (the first index on ties); the pad is excluded
        const int c = threadIdx.x;
        const double tc = A[c][c];
        int rank = 0;
        for (int d = 0; d < b; ++d) rank += (A[d][d] > tc || (A[d][d] == tc && d < c)) ? 1 : 0;
        perm[rank] = c;
        theta[rank] = tc;
    }
    __syncthreads();
    // V2 = V Q, W2 = W Q: element (c, l), consecutive l per lane
    const int lp = (n + 63) & ~63;
    for (int e = threadIdx.x; e < b * lp; e += kPcaBlock) {
        const int c = e / lp, l = e % lp;
        if (l < n) {
            const int pc = perm[c];
            double sv = 0.0, sw = 0.0;
            for (int a = 0; a < b; ++a) {
                const double qa = Q[a][pc];
                sv = __builtin_fma(V[(int64_t)a * ld + l], qa, sv);
                sw = __builtin_fma(W[(int64_t)a * ld + l], qa, sw);
            }
            V2[(int64_t)c * ld + l] = sv;
            W2[(int64_t)c * ld + l] = sw;
        }
    }
    __syncthreads();
    // residuals of the first k <= 16 Ritz pairs: a wavefront each
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double r = 0.0;
    if (w < k)
        for (int l = lane; l < n; l += kWave) {
            const double d = W2[(int64_t)w * ld + l] - theta[w] * V2[(int64_t)w * ld + l];
            r = __builtin_fma(d, d, r);
        }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) r += __shfl_xor(r, o, kWave);
    if (lane == 0) res[w] = sqrt(r);
    __syncthreads();
    if (threadIdx.x == 0) {
        double mx = 0.0;
        for (int c = 0; c < k; ++c) mx = fmax(mx, res[c]);
        out[b] = theta[0] > 0.0 ? mx / theta[0] : 0.0;
    }
    if (threadIdx.x < b) out[threadIdx.x] = theta[threadIdx.x];
}

// P (n x k row-major) from the first k columns of V, each column's
// largest-magnitude component made positive (the first on ties).  A block of
// one wavefront per column.
__global__ __launch_bounds__(64) void k_pca_out(const double *__restrict__ V, int n, int k, int ld,
                                                double *__restrict__ P) {
    const int c = blockIdx.x, lane = threadIdx.x;
    const double *v = V + (int64_t)c * ld;
    int t = 0x7fffffff;
    double mx = -1.0;
    for (int l = lane; l < n; l += kWave)
        if (fabs(v[l]) > mx) { mx = fabs(v[l]); t = l; }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double m2 = __shfl_xor(mx, o, kWave);
        const int t2 = __shfl_xor(t, o, kWave);
        if (m2 > mx || (m2 == mx && t2 < t)) { mx = m2; t = t2; }
    }
    const double sgn = t < n && v[t] < 0.0 ? -1.0 : 1.0;
    for (int l = lane; l < n; l += kWave) P[(int64_t)l * k + c] = sgn * v[l];
}

}  // namespace sap
