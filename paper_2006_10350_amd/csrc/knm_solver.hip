// Preconditioner, preconditioned operator, conjugate gradient and predictor (Alg. 1).
//
// Everything here is fp64 and runs once per fit or is O(M^2) per iteration; the
// O(n M) work of every iteration is the fp32 kernel product of the sweep engines.
// T and A are upper triangular with T^T T = K_MM + jitter I and A^T A = T T^T / M + lambda I
// (Eq. 7 with K_mm = T^T T).  Both live in ONE column-major array of leading dimension ld = M + 2
// (M + 3 for odd M), as in the paper's in-place preconditioner (Sec. 3.1, the figure of the memory
// layout): T in the upper triangle, T(r, c) at r + c ld, and the transpose of A two rows below the
// diagonal, A(r, c) at 2 + c + r ld (a lower triangle; the two rows keep both diagonals and leave
// every column 16-byte aligned).  Code that works on either factor addresses entry (r, c), r <= c,
// of an upper factor R as base[r + c ld] ("upper storage") or base[c + r ld] ("lower storage").
// The factorisations are the block
// column update of Sec. 4 on the fp64 matrix-core products of knm_dsyrk.hip and a leaf
// kernel; the triangular solves, vector updates and reductions are kernels of this file.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <functional>
#include <new>
#include <type_traits>
#include <vector>

#include "knm_internal.h"
#include "knm_leaf.h"

struct knm_precond {
    int device = 0;
    int64_t M = 0;
    double lambda = 0.0, jitter = 0.0;
    double *buf = nullptr; // the shared array, ld x M doubles
    int64_t ld = 0;
    double *T = nullptr;   // = buf: upper storage
    double *A = nullptr;   // = buf + 2: lower storage (what is in memory is A^T, a lower triangle)
    // inverses of the sb x sb diagonal blocks of T and A (column-major blocks, each mirrored onto
    // its lower triangle, the last one padded with the identity), used by the blocked
    // triangular solves; xw (4 M kSolveCols entries) holds the solution, and for several columns the right-hand side, of a
    // solve under way
    int sb = 0;
    double *Tdinv = nullptr;
    double *Adinv = nullptr;
    double *xw = nullptr;
    // sb x sb doubles for the solves with many right-hand sides (one block inverse with its mirror image
    // cleared); null for small M
    double *blk = nullptr;
    // context whose pool the arrays came from (a fit's own preconditioner), null if they are the object's own
    knm_ctx *pool = nullptr;
};

namespace {

using namespace knm;

// Upper triangle (column-major with leading dimension ldk, r <= c) of K[r, c] = k(c_r, c_c) + jitter [r == c], fp64, direct
// differences: k = exp(-|c_r - c_c|^2 scale) with scale = 1 / (2 sigma^2) for the Gaussian kernel; for the
// kernels of r = |c_r - c_c|, with u = r scale: exp(-u), scale = 1 / sigma (Laplacian);
// (1 + u) exp(-u), scale = sqrt(3) / sigma; (1 + u + u^2 / 3) exp(-u), scale = sqrt(5) / sigma (Matern).  The factorisation reads nothing below the diagonal.
// One workgroup of 16 x 16 threads per 64 x 64 tile on or above the diagonal; thread (tx, ty) owns the entries
// (r0 + tx + 16 i, c0 + ty + 16 j), i, j < 4.  The rows of both sides are staged through LDS 16 features at a
// time as doubles, feature-major, so that the 16 threads of a row of the block read consecutive words; every
// squared distance is summed over the features in their order.
constexpr int kKmmTile = 64;
constexpr int kKmmChunk = 16;
__global__ __launch_bounds__(256) void kmm_kernel(const float *__restrict__ C, int64_t M, int d, int64_t ldc, int kind,
                                                  double scale, double jitter, double *__restrict__ K, int64_t ldk)
{
    if (blockIdx.x > blockIdx.y) return; // tile below the diagonal
    __shared__ double rows_r[kKmmChunk][kKmmTile];
    __shared__ double rows_c[kKmmChunk][kKmmTile];
    const int tid = threadIdx.x;
    const int tx = tid & 15, ty = tid >> 4;
    const int64_t r0 = (int64_t)blockIdx.x * kKmmTile, c0 = (int64_t)blockIdx.y * kKmmTile;
    // staging role: row tid / 4 of the tile, features 4 (tid % 4) .. + 3 of the chunk
    const int srow = tid >> 2, sf = (tid & 3) * 4;
    const bool in_r = r0 + srow < M, in_c = c0 + srow < M;
    const float *pr = C + (in_r ? r0 + srow : 0) * ldc;
    const float *pc = C + (in_c ? c0 + srow : 0) * ldc;
    double s[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) s[i][j] = 0.0;
    for (int k0 = 0; k0 < d; k0 += kKmmChunk) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int k = k0 + sf + e;
            const bool kin = k < d;
            rows_r[sf + e][srow] = (in_r && kin) ? (double)pr[kin ? k : 0] : 0.0;
            rows_c[sf + e][srow] = (in_c && kin) ? (double)pc[kin ? k : 0] : 0.0;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kKmmChunk; ++k) {
            double a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = rows_r[k][tx + 16 * i];
#pragma unroll
            for (int j = 0; j < 4; ++j) b[j] = rows_c[k][ty + 16 * j];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const double diff = a[i] - b[j];
                    s[i][j] += diff * diff;
                }
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t r = r0 + tx + 16 * i, c = c0 + ty + 16 * j;
            if (r > c || c >= M) continue;
            double v;
            if (kind == KNM_KERNEL_GAUSSIAN) {
                v = exp(-s[i][j] * scale);
            } else {
                const double u = sqrt(s[i][j]) * scale;
                const double poly = kind == KNM_KERNEL_MATERN32 ? 1.0 + u : kind == KNM_KERNEL_MATERN52 ? 1.0 + u + u * u / 3.0 : 1.0;
                v = poly * exp(-u);
            }
            if (r == c) v += jitter;
            K[r + c * ldk] = v;
        }
}

// row-major (rows x t, leading dimension t) float  <->  column-major (rows x t) double
__global__ void f32_rows_to_f64_cols(const float *__restrict__ src, int64_t rows, int t, double *__restrict__ dst)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= rows * t) return;
    const int64_t r = i / t;
    const int c = (int)(i % t);
    dst[r + (int64_t)c * rows] = (double)src[i];
}
__global__ void f64_cols_to_f32_rows(const double *__restrict__ src, int64_t rows, int t, float *__restrict__ dst)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= rows * t) return;
    const int64_t r = i / t;
    const int c = (int)(i % t);
    dst[i] = (float)src[r + (int64_t)c * rows];
}
__global__ void f64_rows_to_cols(const double *__restrict__ src, int64_t rows, int t, double *__restrict__ dst, int back)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= rows * t) return;
    const int64_t r = i / t;
    const int c = (int)(i % t);
    if (back) dst[i] = src[r + (int64_t)c * rows];
    else dst[r + (int64_t)c * rows] = src[i];
}

// dst[r * cols + c] = entry (row0 + r, col0 + c) of an upper factor stored at F (upper or lower storage,
// leading dimension ld), zero below the diagonal: a block of a factor gathered into row-major order
__global__ void gather_block_kernel(const double *__restrict__ F, int64_t ld, int lower, int64_t row0, int64_t col0,
                                    int64_t rows, int64_t cols, double *__restrict__ dst)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= rows * cols) return;
    const int64_t r = row0 + i / cols, c = col0 + i % cols;
    dst[i] = (c >= r) ? (lower ? F[c + r * ld] : F[r + c * ld]) : 0.0;
}

// ---- blocked triangular solves -----------------------------------------------------------------
// R (upper, column-major, leading dimension M) is cut into block columns of width sb.  A solve
// walks the diagonal blocks in dependency order; each step multiplies a right-hand-side block
// by the pre-inverted diagonal block and then updates the remaining right-hand side with the
// off-diagonal panel, which is streamed once with coalesced loads.  The panels are ~all of
// the 8 M^2 / 2 bytes of the factor, so a solve is bound by HBM bandwidth; wide blocks keep the
// chain of dependent launches short (M / sb steps) and every launch large enough to fill the
// chip.
//
// Each inverted diagonal block is stored mirrored: S[i, j] = S[j, i] = inv(R_kk)[min, max].  Both
// the plain and the transposed product then read contiguous pieces of the columns of S.
// Blocks of at most 2048, all about as wide: up to M = 2048 a solve is one product with the whole inverse.
// Forming the inverses costs M sb^2 flop, next to the M^3 of the factorisations; narrower blocks (M / 16) made a
// solve a chain of 32 launches at any M.
// Precision: errors against extended precision, in units of those of substitution in fp64 (M = 1000 to 4500, jitter 1e-8 and 0, pivots
// in ratios up to 7e4): 0.6 to 1.2, 2.2 for the transposed solve with one block of 2000 and a pivot ratio of 9e3.  Blocks of
// 1024: 0.5 to 1.7, fits 0 to 3 % slower (M = 10k, 10 columns: 132.5 -> 136.3 ms); 512: 0.4 to 1.0, 5 to 18 % slower; M / 16: 0.3
// to 0.6.  All of it is rounding of 1e-15 where the products of a fit leave 1e-7.
inline int solve_block_width(int64_t M)
{
    const int64_t blocks = (M + 2047) / 2048;
    return (int)(((M + blocks - 1) / blocks + 127) / 128 * 128);
}

// copy the upper triangle of every block onto its strict lower triangle
__global__ void mirror_upper_kernel(double *__restrict__ S, int sb)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x; // row in the lower triangle
    const int j = blockIdx.y;                            // column
    if (i >= sb || i <= j) return;
    double *blk = S + (int64_t)blockIdx.z * sb * sb;
    blk[i + (int64_t)j * sb] = blk[j + (int64_t)i * sb];
}

__device__ __forceinline__ double wave_sum(double s)
{
    s += __shfl_xor(s, 32);
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 8);
    s += __shfl_xor(s, 4);
    s += __shfl_xor(s, 2);
    s += __shfl_xor(s, 1);
    return s;
}

typedef double solve_d2 __attribute__((ext_vector_type(2)));

// One right-hand side: the three kernels below, bound by the bandwidth of the factor.

// x = inv(R_kk) b (lower = 1: x[c] = sum_{i >= c} S[i, c] b[i]) or x = inv(R_kk)^T b (lower = 0:
// x[c] = sum_{i <= c} S[i, c] b[i]) for one mirrored block S of live order nbk; one wavefront
// per entry of x, lanes along the column of S, 1024 entries of it in flight (with two 8-byte loads per lane in flight a block of
// 2048 took 10.9 us).  sb even, S 16-byte aligned.  Where they are given: sum[c] = x[c] + scale add[c], x32[c] = x[c] rounded.
__global__ __launch_bounds__(256) void diag_apply_kernel(const double *__restrict__ S, int sb, int nbk, int lower,
                                                        const double *__restrict__ b, double *__restrict__ x,
                                                        const double *__restrict__ add, double scale,
                                                        double *__restrict__ sum, float *__restrict__ x32)
{
    const int lane = threadIdx.x & 63;
    const int c = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (c >= nbk) return;
    const double *col = S + (int64_t)c * sb;
    const int lo = lower ? c : 0;
    const int hi = lower ? nbk : c + 1;
    constexpr int kFlight = 8;
    double s0 = 0.0, s1 = 0.0;
    for (int i0 = (lo & ~1) + 2 * lane; i0 < hi; i0 += 128 * kFlight) {
        solve_d2 a[kFlight];
        double b0[kFlight], b1[kFlight];
#pragma unroll
        for (int u = 0; u < kFlight; ++u) { // (an entry outside the range is taken from the column's first pair and dropped)
            const int i = i0 + 128 * u, ia = i < hi ? i : 0;
            a[u] = *reinterpret_cast<const solve_d2 *>(col + ia);
            b0[u] = b[ia];
            b1[u] = b[ia + 1 < nbk ? ia + 1 : 0];
        }
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            const int i = i0 + 128 * u;
            if (i >= lo && i < hi) s0 = fma(a[u][0], b0[u], s0);
            if (i + 1 < hi) s1 = fma(a[u][1], b1[u], s1);
        }
    }
    const double s = wave_sum(s0 + s1);
    if (lane == 0) {
        x[c] = s;
        if (sum != nullptr) sum[c] = s + scale * add[c];
        if (x32 != nullptr) x32[c] = (float)s;
    }
}

constexpr int kPanelWaves = 16; // wavefronts of a panel_update_n workgroup, sharing the columns
// Rows of a panel_update_n workgroup: 32, and 16 up to this many, which would be at most 64 workgroups of 32 (2048 x 2048: 17.7 -> 12.9 us; 4096 rows
// the same, 6144 21.9 -> 29.5).
constexpr int64_t kPanelShortUpTo = 2048;

// b[r] = src[r] - sum_j P[r + (k0 + j) ld] x[j] for r in [r_lo, r_hi)  (x = the solved block, nbk entries; src: the
// right-hand side so far, b itself from the second block on): the rows above the block of an upper-storage factor
// in its plain solve, the rows below the block of a lower-storage factor in its transposed solve.  ld and r_lo even, R 16-byte
// aligned, column entries up to the next even row readable.  ROWS / 2 lanes take ROWS rows of a column, the lane groups of
// 16 wavefronts 64 columns (of 32 rows) at a time, eight loads in flight each: with 64 rows per workgroup of 8 wavefronts an update of 3000 rows
// had 46 workgroups.
template <int ROWS>
__global__ __launch_bounds__(kPanelWaves * 64) void panel_update_n_kernel(const double *__restrict__ R, int64_t M,
                                                                         int64_t k0, int nbk, int64_t r_lo,
                                                                         int64_t r_hi, const double *__restrict__ x,
                                                                         const double *src, double *b)
{
    __shared__ double part[kPanelWaves][ROWS];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    constexpr int kLanes = ROWS / 2, kGroups = 64 / kLanes; // lanes along a column, columns at a time
    const int l = lane % kLanes, q = lane / kLanes;
    const int64_t r = r_lo + (int64_t)blockIdx.x * ROWS + 2 * l;
    const double *p = R + (r < r_hi ? r : r_lo) + k0 * M;
    constexpr int kStep = kGroups * kPanelWaves;
    double s0 = 0.0, s1 = 0.0;
    for (int j0 = kGroups * w + q; j0 < nbk; j0 += 8 * kStep) {
        solve_d2 a[8];
        double xv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int j = j0 + u * kStep, jc = j < nbk ? j : j0;
            a[u] = *reinterpret_cast<const solve_d2 *>(p + (int64_t)jc * M);
            xv[u] = x[jc];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (j0 + u * kStep < nbk) {
                s0 = fma(a[u][0], xv[u], s0);
                s1 = fma(a[u][1], xv[u], s1);
            }
    }
#pragma unroll
    for (int m = 32; m >= kLanes; m >>= 1) {
        s0 += __shfl_xor(s0, m);
        s1 += __shfl_xor(s1, m);
    }
    if (q == 0) {
        part[w][2 * l] = s0;
        part[w][2 * l + 1] = s1;
    }
    __syncthreads();
    const int64_t row = r_lo + (int64_t)blockIdx.x * ROWS + threadIdx.x;
    if (threadIdx.x < ROWS && row < r_hi) {
        double s = 0.0;
#pragma unroll
        for (int u = 0; u < kPanelWaves; ++u) s += part[u][threadIdx.x];
        b[row] = src[row] - s;
    }
}

// b[j] = src[j] - sum_i P[(k0 + i) + j ld] x[i] for j in [j0, j1)  (x = the solved block, nbk entries): the
// columns right of the block of an upper-storage factor in its transposed solve, the columns left of
// the block of a lower-storage factor in its plain solve.  One wavefront per column, lanes along the rows, 1024 entries in flight as in
// diag_apply_kernel; R 16-byte aligned, ld and k0 even, column entries up to the next even row readable.  Four columns per wavefront, 8-byte loads
// of 256 entries of each in flight, were too few wavefronts for a short panel (2048 x 2048 14.3 us, 8.7 now; 2048 x 10240 37.1, 32.3) and no faster
// for a long one.
__global__ __launch_bounds__(256) void panel_update_t_kernel(const double *__restrict__ R, int64_t M, int64_t k0, int nbk, int64_t j0, int64_t j1,
                                                                  const double *__restrict__ x, const double *src, double *b)
{
    const int lane = threadIdx.x & 63;
    const int64_t j = j0 + (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (j >= j1) return;
    const double *p = R + k0 + j * M;
    constexpr int kFlight = 8;
    double s0 = 0.0, s1 = 0.0;
    for (int i0 = 2 * lane; i0 < nbk; i0 += 128 * kFlight) {
        solve_d2 a[kFlight];
        double x0[kFlight], x1[kFlight];
#pragma unroll
        for (int u = 0; u < kFlight; ++u) { // (an entry past the end is taken from the column's first pair and dropped)
            const int i = i0 + 128 * u, ia = i < nbk ? i : 0;
            a[u] = *reinterpret_cast<const solve_d2 *>(p + ia);
            x0[u] = x[ia];
            x1[u] = x[ia + 1 < nbk ? ia + 1 : 0];
        }
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            const int i = i0 + 128 * u;
            if (i < nbk) s0 = fma(a[u][0], x0[u], s0);
            if (i + 1 < nbk) s1 = fma(a[u][1], x1[u], s1);
        }
    }
    const double s = wave_sum(s0 + s1);
    if (lane == 0) b[j] = src[j] - s;
}

// 2 to 16 right-hand sides: the same steps as skinny products on the fp64 matrix cores, still bound by the
// bandwidth of the factor, which is read once for all columns (a 16 x 16 x 4 instruction takes 512 bytes of it in 64
// cycles: 19 TB/s over the chip).  Right-hand sides and solution live as [row][16] arrays, unused columns zero.
// 10 columns at M = 10000: 5.2 ms for the four solves of an iteration as vector-ALU passes over 8 and 2 columns,
// 1.07 ms with 32 outputs and 8 wavefronts per workgroup (62 to 250 workgroups of a panel, 64 of a diagonal block), 0.83 ms with 16 of either, 0.70 ms now.
constexpr int kSolveCols = 16;
constexpr int kSkinnyThreads = 1024, kSkinnyWaves = kSkinnyThreads / 64;
typedef double solve_d4 __attribute__((ext_vector_type(4)));
// Outputs of a workgroup, whose 16 wavefronts share the contraction 32 at a time: 16 NT.  A product of at most 2048
// outputs (a diagonal block) is 128 workgroups with NT = 1.
constexpr int64_t kSkinnyNarrowUpTo = 2048;
// Up to this many such workgroups two share the contraction, each with its own part of the sums (`half` entries apart), so that
// they fill the chip: every right-hand side and solution of a solve is the sum of two parts, which its readers form, always in that order.
// M = 10000: diagonal block 16.1 -> 12.3 us, panel of 2000 rows 17.8 -> 13.8, of 4000 rows 24.0 -> 19.9 and 32.2 -> 23.1; of
// 6000 rows (two each on half of the CUs) 26 -> 34.
constexpr unsigned kSkinnySplitUpTo = 128;

// adds up the wavefronts' accumulators; this thread's entry of the tile (threads below 256 NT): accumulator t = tid / 256,
// register (tid / 64) % 4 of lane tid % 64
template <int NT> __device__ __forceinline__ double skinny_reduce(double (*red)[NT][4][64], const solve_d4 (&acc)[NT])
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave][t][r][lane] = acc[t][r];
    __syncthreads();
    double s = 0.0;
    if (tid < 256 * NT) {
#pragma unroll
        for (int w = 0; w < kSkinnyWaves; ++w) s += red[w][tid >> 8][(tid >> 6) & 3][lane];
    }
    return s;
}

// b[r, c] -= sum_{k < nk} P[r + k ld] x[k, c], r < rows.  P 16-byte aligned, ld even, and column entries up to the next
// even row readable.  A lane's load of NT entries holds the same column entry of rows NT l ... NT l + NT - 1: accumulator t
// has rows t mod NT.
template <int NT>
__global__ __launch_bounds__(kSkinnyThreads) void skinny_n_kernel(const double *__restrict__ P, int64_t ld, int64_t rows,
                                                                 int nk, const double *__restrict__ x, double *__restrict__ b,
                                                                 int64_t half)
{
    typedef double row_t __attribute__((ext_vector_type(NT)));
    __shared__ double red[kSkinnyWaves][NT][4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l15 = lane & 15, q = lane >> 4;
    const int step = kSkinnyWaves * 32 * (int)gridDim.y;
    const int64_t row0 = (int64_t)blockIdx.x * (16 * NT);
    const double *p = P + (row0 + NT * l15 < rows ? row0 + NT * l15 : 0);
    solve_d4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = solve_d4{0.0, 0.0, 0.0, 0.0};
    for (int k0 = ((int)blockIdx.y * kSkinnyWaves + wave) * 32; k0 < nk; k0 += step) {
        row_t a[8];
        double bv[8], b2[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int k = k0 + 4 * s + q, kc = k < nk ? k : nk - 1;
            a[s] = *reinterpret_cast<const row_t *>(p + (int64_t)kc * ld);
            bv[s] = x[(int64_t)kc * kSolveCols + l15];
            b2[s] = x[half + (int64_t)kc * kSolveCols + l15];
        }
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const bool in = k0 + 4 * s + q < nk;
            const double bs = in ? bv[s] + b2[s] : 0.0;
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? a[s][t] : 0.0, bs, acc[t], 0, 0, 0);
        }
    }
    const double s = skinny_reduce<NT>(red, acc);
    const int t = threadIdx.x >> 8, i = 4 * ((threadIdx.x >> 6) & 3) + q;
    const int64_t r = row0 + NT * i + t;
    if (t < NT && r < rows) b[blockIdx.y * half + r * kSolveCols + l15] -= s;
}

// MODE 0: b[j, c] -= sum_{i < nk} P[i + j ld] x[i, c], j < outs.  MODE 1, 2: b[j, c] = the same sum over i >= j, i <= j (a
// mirrored block inverse: the plain and the transposed solve with its diagonal block).  P 16-byte aligned, ld even.  A
// lane holds 8 consecutive i of its column, 32 per 4 lane groups.
template <int MODE, int NT>
__global__ __launch_bounds__(kSkinnyThreads) void skinny_t_kernel(const double *__restrict__ P, int64_t ld, int64_t outs,
                                                                 int nk, const double *__restrict__ x, double *__restrict__ b,
                                                                 int64_t half)
{
    __shared__ double red[kSkinnyWaves][NT][4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l15 = lane & 15, q = lane >> 4;
    const int64_t tile0 = (int64_t)blockIdx.x * (16 * NT);
    const double *p[NT];
    solve_d4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int64_t j = tile0 + 16 * t + l15;
        p[t] = P + (j < outs ? j : 0) * ld;
        acc[t] = solve_d4{0.0, 0.0, 0.0, 0.0};
    }
    const int first = MODE == 1 ? (int)tile0 & ~31 : 0;
    const int last = MODE == 2 && tile0 + 16 * NT < nk ? (int)tile0 + 16 * NT : nk;
    const int step = kSkinnyWaves * 32 * (int)gridDim.y;
    for (int i0 = first + ((int)blockIdx.y * kSkinnyWaves + wave) * 32; i0 < last; i0 += step) {
        solve_d2 a[NT][4];
        double bv[8], b2[8];
        const int ib = i0 + 8 * q; // nk and ld are such that 8 entries from an in-range multiple of 8 stay inside the array
        const bool any = ib < nk;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int i = any && ib + 2 * s < nk ? ib + 2 * s : 0;
                a[t][s] = *reinterpret_cast<const solve_d2 *>(p[t] + i);
            }
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int64_t at = (int64_t)(ib + s < nk ? ib + s : 0) * kSolveCols + l15;
            bv[s] = x[at];
            b2[s] = x[half + at];
        }
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int i = ib + s;
            const double bs = i < nk ? bv[s] + b2[s] : 0.0;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int j = (int)tile0 + 16 * t + l15;
                const bool in = i < nk && (MODE == 0 || (MODE == 1 ? i >= j : i <= j));
                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? a[t][s >> 1][s & 1] : 0.0, bs, acc[t], 0, 0, 0);
            }
        }
    }
    const double s = skinny_reduce<NT>(red, acc);
    const int t = threadIdx.x >> 8;
    const int64_t j = tile0 + 16 * t + 4 * ((threadIdx.x >> 6) & 3) + q;
    if (t < NT && j < outs) {
        double *const out = b + blockIdx.y * half + j * kSolveCols + l15;
        if (MODE == 0) *out -= s;
        else *out = s;
    }
}

// [row][16] <- tc columns of a column-major array (zero from tc on), and back
__global__ void cols_to_rows16_kernel(const double *__restrict__ B, int64_t ldb, int64_t M, int tc, double *__restrict__ out, int64_t half)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t r = e % M;
    const int c = (int)(e / M);
    if (c >= kSolveCols) return;
    out[r * kSolveCols + c] = c < tc ? B[(int64_t)c * ldb + r] : 0.0;
    out[half + r * kSolveCols + c] = 0.0;
}
// (with add: plus scale add, same layout as B)
__global__ void rows16_to_cols_kernel(const double *__restrict__ in, int64_t half, int64_t M, int tc, double *__restrict__ B, int64_t ldb,
                                      const double *__restrict__ add, double scale)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t r = e % M;
    const int c = (int)(e / M);
    if (c < tc)
        B[(int64_t)c * ldb + r] = (in[r * kSolveCols + c] + in[half + r * kSolveCols + c]) + (add != nullptr ? scale * add[(int64_t)c * ldb + r] : 0.0);
}

__global__ __launch_bounds__(kLeafThreads) void potrf_trtri_leaf_kernel(LeafArgs l)
{
    __shared__ double sh[kLeafDoubles];
    leaf_block(l, sh);
}

inline dim3 grid1(int64_t n, int threads = 256) { return dim3((unsigned)((n + threads - 1) / threads)); }

// ---- fp64 vector work of the CG driver -----------------------------------------------------
// Every sum is a fixed number of block partials, added up in a fixed order by each block of the kernel that
// needs the total, so a fit repeats itself bit for bit (where the card has room for what is for speed alone, or never has).  The scalars of CG stay on the device: an iteration takes three
// launches for all columns and the host never waits (with the two scalars of a column read back and five launches per
// column, 10 columns cost 50 launches and 20 synchronisations per iteration: 0.5 ms of the 4.4 ms at
// n = 60k, M = 10k).
constexpr int kMaxRedBlocks = 64;
inline int red_blocks(int64_t M)
{
    const int64_t b = (M + 1023) / 1024;
    return (int)(b < kMaxRedBlocks ? b : kMaxRedBlocks);
}

// sum over the 256 threads of a block, in every thread
__device__ __forceinline__ double block_sum(double s, double *sh)
{
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}
// total of the `count` <= 64 partials of a vector, in every thread
__device__ __forceinline__ double partials_sum(const double *__restrict__ part, int count)
{
    const int lane = threadIdx.x & 63;
    return wave_sum(lane < count ? part[lane] : 0.0);
}

// part[c][block] <- this block's share of sum_i x[i, c] y[i, c] (y null: of sum_i x[i, c])
__global__ __launch_bounds__(256) void dot_partial_kernel(const double *__restrict__ x, const double *__restrict__ y,
                                                         int64_t M, double *__restrict__ part)
{
    __shared__ double sh[4];
    const int64_t c = blockIdx.y;
    double s = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < M; i += (int64_t)gridDim.x * 256)
        s += y ? x[c * M + i] * y[c * M + i] : x[c * M + i];
    s = block_sum(s, sh);
    if (threadIdx.x == 0) part[c * gridDim.x + blockIdx.x] = s;
}

// out[c] <- scale times the total of the partials of column c = blockIdx.x
__global__ __launch_bounds__(64) void dot_finish_kernel(const double *__restrict__ part, int count, double scale,
                                                       double *__restrict__ out)
{
    const double s = partials_sum(part + (int64_t)blockIdx.x * count, count);
    if (threadIdx.x == 0) out[blockIdx.x] = scale * s;
}

// a = rho / (p . q); b += a p; r -= a q; part_rr <- partials of the new r . r
__global__ __launch_bounds__(256) void cg_step_kernel(int64_t M, const double *__restrict__ rho, const double *__restrict__ part_pq,
                                                     const double *__restrict__ p, const double *__restrict__ q,
                                                     double *__restrict__ b, double *__restrict__ r, double *__restrict__ part_rr)
{
    __shared__ double sh[4];
    const int64_t c = blockIdx.y;
    const double pq = partials_sum(part_pq + c * gridDim.x, gridDim.x);
    const double a = (pq != 0.0) ? rho[c] / pq : 0.0;
    double s = 0.0;
    for (int64_t i = c * M + (int64_t)blockIdx.x * 256 + threadIdx.x; i < (c + 1) * M; i += (int64_t)gridDim.x * 256) {
        b[i] += a * p[i];
        const double v = r[i] - a * q[i];
        r[i] = v;
        s += v * v;
    }
    s = block_sum(s, sh);
    if (threadIdx.x == 0) part_rr[c * gridDim.x + blockIdx.x] = s;
}

// rho_next = r . r; p = r + (rho_next / rho) p
__global__ __launch_bounds__(256) void cg_direction_kernel(int64_t M, const double *__restrict__ rho, double *__restrict__ rho_next,
                                                          const double *__restrict__ part_rr, const double *__restrict__ r,
                                                          double *__restrict__ p)
{
    const int64_t c = blockIdx.y;
    const double rn = partials_sum(part_rr + c * gridDim.x, gridDim.x);
    const double b = (rho[c] != 0.0) ? rn / rho[c] : 0.0;
    for (int64_t i = c * M + (int64_t)blockIdx.x * 256 + threadIdx.x; i < (c + 1) * M; i += (int64_t)gridDim.x * 256)
        p[i] = r[i] + b * p[i];
    if (blockIdx.x == 0 && threadIdx.x == 0) rho_next[c] = rn;
}

// All three steps after an application of the operator, one workgroup per column, for M up to kCgAtOnce: 1024 blocks entries, four per
// thread, in the same partials and order as dot_partial_kernel, cg_step_kernel and cg_direction_kernel.  Bound by latency: M = 1000 5 us in place of 9
// and two gaps between launches.  Longer vectors are more than a CU brings in as fast as the chip.
constexpr int64_t kCgAtOnce = 4096;
__global__ __launch_bounds__(1024) void cg_update_kernel(int64_t M, const double *__restrict__ rho, double *__restrict__ rho_next,
                                                        double *__restrict__ p, const double *__restrict__ q, double *__restrict__ b,
                                                        double *__restrict__ r)
{
    __shared__ double sh[2][4][4], part[2][4];
    const int64_t c = blockIdx.x;
    const int wave = threadIdx.x >> 6, blocks = blockDim.x >> 8;
    double pv[4], qv[4], rv[4], bv[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int64_t i = threadIdx.x + (int64_t)blockDim.x * k, j = c * M + (i < M ? i : 0);
        pv[k] = p[j];
        qv[k] = q[j];
        rv[k] = r[j];
        bv[k] = b[j];
    }
    auto total = [&](int which, double s) { // of every thread's s, as block_sum and partials_sum have it
        s = wave_sum(s);
        if ((threadIdx.x & 63) == 0) sh[which][wave >> 2][wave & 3] = s;
        __syncthreads();
        const double *const w = sh[which][threadIdx.x & 3];
        if (threadIdx.x < (unsigned)blocks) part[which][threadIdx.x] = (w[0] + w[1]) + (w[2] + w[3]);
        __syncthreads();
        return partials_sum(part[which], blocks);
    };
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (threadIdx.x + (int64_t)blockDim.x * k < M) s += pv[k] * qv[k];
    const double pq = total(0, s);
    const double a = (pq != 0.0) ? rho[c] / pq : 0.0;
    s = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        rv[k] = rv[k] - a * qv[k];
        if (threadIdx.x + (int64_t)blockDim.x * k < M) s += rv[k] * rv[k];
    }
    const double rn = total(1, s);
    const double e = (rho[c] != 0.0) ? rn / rho[c] : 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int64_t i = threadIdx.x + (int64_t)blockDim.x * k;
        if (i >= M) continue;
        b[c * M + i] = bv[k] + a * pv[k];
        r[c * M + i] = rv[k];
        p[c * M + i] = rv[k] + e * pv[k];
    }
    if (threadIdx.x == 0) rho_next[c] = rn;
}

// The steps of CG after an application of the operator: q = H p in hand, rho = r . r
void launch_cg_update(hipStream_t stream, int64_t M, int t, const double *rho, double *rho_next, double *p, const double *q, double *b, double *r,
                      double *part_pq, double *part_rr)
{
    const int blocks = red_blocks(M);
    const dim3 vgrid((unsigned)blocks, (unsigned)t), vblock(256);
    if (M <= kCgAtOnce) {
        hipLaunchKernelGGL(cg_update_kernel, dim3((unsigned)t), dim3(256u * blocks), 0, stream, M, rho, rho_next, p, q, b, r);
        return;
    }
    hipLaunchKernelGGL(dot_partial_kernel, vgrid, vblock, 0, stream, p, q, M, part_pq);
    hipLaunchKernelGGL(cg_step_kernel, vgrid, vblock, 0, stream, M, rho, part_pq, p, q, b, r, part_rr);
    hipLaunchKernelGGL(cg_direction_kernel, vgrid, vblock, 0, stream, M, rho, rho_next, part_rr, r, p);
}

// y32 <- (y += x) rounded
__global__ void add_round_kernel(int64_t n, const double *__restrict__ x, double *__restrict__ y, float *__restrict__ y32)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double v = y[i] + x[i];
    y[i] = v;
    y32[i] = (float)v;
}

// Logistic loss l(z, y) = log(1 + exp(-y z)), y = +-1 (Appendix "Logistic Falkon Algorithm",
// Example 1a), evaluated in fp64 from fp32 predictions: first derivative g, second derivative
// dw (as float for the sweeps and/or as double for the preconditioner), loss.  Any output may
// be null.
__global__ void logistic_terms_kernel(const float *__restrict__ z, const float *__restrict__ y, int64_t n,
                                      float *__restrict__ g, float *__restrict__ dw32, double *__restrict__ dw64,
                                      double *__restrict__ loss)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double yi = (double)y[i];
    const double m = yi * (double)z[i];
    const double s = 0.5 * (1.0 - tanh(0.5 * m)); // sigma(-m), stable for either sign
    if (g) g[i] = (float)(-yi * s);
    if (dw32) dw32[i] = (float)(s * (1.0 - s));
    if (dw64) dw64[i] = s * (1.0 - s);
    if (loss) loss[i] = (m > 0.0) ? log1p(exp(-m)) : -m + log1p(exp(m));
}

// r[j] = -(u[j] + c (zc[j] + eps a[j]))   (right-hand side of a Newton step, fp64)
__global__ void newton_rhs_kernel(const float *__restrict__ u, const float *__restrict__ zc,
                                  const double *__restrict__ a, double c, double eps, int64_t M,
                                  double *__restrict__ r)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= M) return;
    r[j] = -((double)u[j] + c * ((double)zc[j] + eps * a[j]));
}

__global__ void axpy_kernel(int64_t n, double a, const double *__restrict__ x, double *__restrict__ y)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] += a * x[i];
}

// Many right-hand sides: the same blocked solve as products on the fp64 matrix cores.
// (two groups of 16 as skinny products still beat them: M = 20000, 32 columns: 6.3 against 7.5 ms for four solves)
constexpr int kProductSolveMinCols = 2 * kSolveCols + 1; // from this many right-hand sides on
constexpr int64_t kProductSolveMinM = 4096; // and this order of the factor

// out <- the upper triangle (diagonal included) of one mirrored block inverse, zeros below it
__global__ void upper_block_kernel(const double *__restrict__ S, int sb, double *__restrict__ out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int c = blockIdx.y;
    if (i < sb) out[i + (int64_t)c * sb] = (i <= c) ? S[i + (int64_t)c * sb] : 0.0;
}

// b[k0 + i + j ldb] = x[i + j ldx], i < nbk, j < tc
__global__ void block_rows_kernel(const double *__restrict__ x, int64_t ldx, int nbk, int tc, double *__restrict__ b,
                                  int64_t ldb)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y;
    if (i < nbk && j < tc) b[i + (int64_t)j * ldb] = x[i + (int64_t)j * ldx];
}

// The blocked solve of tri_solve with both of its steps as products: per block, X = inv(R_kk) B_k or
// inv(R_kk)^T B_k (the block inverse with its mirror image cleared, so that a plain product applies the
// triangular factor), then the rows still to be solved lose the panel times X.  The factor is read once
// per group of columns (as many as the staging array holds: at least 128 from M = 4096 on), at the rate
// of the matrix cores instead of once per 8 columns.
int tri_solve_products(knm_ctx *ctx, const knm_precond *p, const double *R, const double *S, bool trans, double *B, int t)
{
    const int64_t M = p->M, ld = p->ld;
    const bool lower = (R == p->A);
    const int sb = p->sb;
    const int64_t nblk = (M + sb - 1) / sb;
    const int64_t cap = 2 * M * kSolveCols / sb; // columns the staging array holds at leading dimension sb
    double *X = p->xw;
    for (int c0 = 0; c0 < t;) {
        const int tc = (int)((t - c0 < cap) ? t - c0 : cap);
        double *Bc = B + (int64_t)c0 * M;
        for (int64_t step = 0; step < nblk; ++step) {
            const int64_t k = trans ? step : nblk - 1 - step; // R^T is lower: forward; R: backward
            const int64_t k0 = k * sb;
            const int nbk = (int)((M - k0 < sb) ? M - k0 : sb);
            hipLaunchKernelGGL(upper_block_kernel, dim3((unsigned)((sb + 255) / 256), (unsigned)sb), dim3(256), 0, ctx->stream,
                               S + k * sb * sb, sb, p->blk);
            // x[c] = sum_i W[c, i] b[i] (plain) or sum_i W[i, c] b[i] (transposed), W = inv(R_kk) at blk[row + col sb]
            hipError_t e = launch_gemm_f64(trans ? 0 : 1, nbk, tc, nbk, 1.0, p->blk, sb, Bc + k0, M, 0.0, X, sb, ctx->stream);
            if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "triangular solve: block product", e);
            hipLaunchKernelGGL(block_rows_kernel, dim3((unsigned)((nbk + 255) / 256), (unsigned)tc), dim3(256), 0, ctx->stream, X,
                               (int64_t)sb, nbk, tc, Bc + k0, M);
            // the rows of B still to be solved: before the block (plain) or after it (transposed)
            const int64_t lo = trans ? k0 + nbk : 0, hi = trans ? M : k0;
            if (hi > lo) {
                // panel entry (row r of the rest, column kk of the block): R[r + (k0 + kk) ld] where the panels
                // are contiguous in r, else R[(k0 + kk) + r ld]
                e = (trans == lower)
                        ? launch_gemm_f64(1, hi - lo, tc, nbk, -1.0, R + lo + k0 * ld, ld, X, sb, 1.0, Bc + lo, M, ctx->stream)
                        : launch_gemm_f64(0, hi - lo, tc, nbk, -1.0, R + k0 + lo * ld, ld, X, sb, 1.0, Bc + lo, M, ctx->stream);
                if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "triangular solve: panel product", e);
            }
        }
        c0 += tc;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "blocked triangular solve", e);
    return KNM_OK;
}

// out <- op(R)^-1 in + scale add for column-major M x t arrays; S = mirrored inverses of the diagonal blocks of R
// (R = p->T, upper storage, or p->A, lower storage); add may be null; with one column out32, where it is given, receives the
// solution (without add) rounded.  `in` and `out` must not overlap for one column.  p->xw holds the solve's
// intermediate vectors; solves on one context are stream-ordered.  Either storage streams its panels along contiguous columns
// of the array: what is a row update for one is a column update for the other.
int tri_solve(knm_ctx *ctx, const knm_precond *p, const double *R, const double *S, bool trans, const double *in, double *out, int t,
              const double *add = nullptr, double scale = 0.0, float *out32 = nullptr)
{
    TraceRange range(R == p->A ? (trans ? "knm solve A^-T" : "knm solve A^-1") : (trans ? "knm solve T^-T" : "knm solve T^-1"));
    const int64_t M = p->M, ld = p->ld;
    const bool lower = (R == p->A);
    const int sb = p->sb;
    const int64_t nblk = (M + sb - 1) / sb;
    if (t >= kProductSolveMinCols && p->blk != nullptr) {
        if (in != out && hipMemcpyAsync(out, in, sizeof(double) * M * t, hipMemcpyDeviceToDevice, ctx->stream) != hipSuccess)
            return fail(ctx, KNM_HIP_ERROR, "triangular solve: copy");
        int st = tri_solve_products(ctx, p, R, S, trans, out, t);
        if (!st && add != nullptr) hipLaunchKernelGGL(axpy_kernel, grid1(M * t), dim3(256), 0, ctx->stream, M * t, scale, add, out);
        return st;
    }
    for (int c0 = 0; c0 < t; c0 += kSolveCols) {
        const int tc = (t - c0 < kSolveCols) ? t - c0 : kSolveCols; // columns that stream the factor together
        const double *bin = in + (int64_t)c0 * M;
        double *bout = out + (int64_t)c0 * M;
        const double *badd = add != nullptr ? add + (int64_t)c0 * M : nullptr;
        const int64_t half = 2 * M * kSolveCols;
        double *rhs = p->xw + M * kSolveCols; // several columns: right-hand side and solution as [row][16] arrays, in two parts each
        if (tc > 1)
            hipLaunchKernelGGL(cols_to_rows16_kernel, grid1(M * kSolveCols), dim3(256), 0, ctx->stream, bin, M, M, tc, rhs, half);
        // one column: the right-hand side so far (`in` up to the first panel update), and where the solution goes
        double *const work = p->xw;
        double *const sol = badd != nullptr ? p->xw + M : bout;
        for (int64_t step = 0; step < nblk; ++step) {
            const int64_t k = trans ? step : nblk - 1 - step; // R^T is lower: forward; R: backward
            const int64_t k0 = k * sb;
            const int nbk = (int)((M - k0 < sb) ? M - k0 : sb);
            const double *Sk = S + k * sb * sb;
            // the entries of b still to be solved: before the block (plain) or after it (transposed)
            const int64_t lo = trans ? k0 + nbk : 0, hi = trans ? M : k0;
            if (tc > 1) {
                double *x = p->xw + k0 * kSolveCols;
                // the diagonal block (of at most 2048, always by two), then the panel of the entries still to be solved
                auto diagonal = [&](auto kernel) {
                    hipLaunchKernelGGL(kernel, dim3((unsigned)((nbk + 15) / 16), 2), dim3(kSkinnyThreads), 0, ctx->stream, Sk, (int64_t)sb,
                                       (int64_t)nbk, nbk, rhs + k0 * kSolveCols, x, half);
                };
                if (trans) diagonal(skinny_t_kernel<2, 1>);
                else diagonal(skinny_t_kernel<1, 1>);
                if (hi == lo) continue;
                const bool narrow = hi - lo <= kSkinnyNarrowUpTo;
                const unsigned tiles = (unsigned)(narrow ? (hi - lo + 15) / 16 : (hi - lo + 31) / 32);
                const dim3 pgrid(tiles, tiles <= kSkinnySplitUpTo ? 2 : 1);
                auto panel = [&](auto kernel, const double *P) {
                    hipLaunchKernelGGL(kernel, pgrid, dim3(kSkinnyThreads), 0, ctx->stream, P, ld, hi - lo, nbk, x, rhs + lo * kSolveCols, half);
                };
                if (trans == lower) // panel entries R(r, k0 + j) or R(k0 + j, r) contiguous in r
                    narrow ? panel(skinny_n_kernel<1>, R + lo + k0 * ld) : panel(skinny_n_kernel<2>, R + lo + k0 * ld);
                else                // contiguous in the block's own index
                    narrow ? panel(skinny_t_kernel<0, 1>, R + k0 + lo * ld) : panel(skinny_t_kernel<0, 2>, R + k0 + lo * ld);
                continue;
            }
            const double *b = step == 0 ? bin : work;
            hipLaunchKernelGGL(diag_apply_kernel, dim3((unsigned)((nbk + 3) / 4)), dim3(256), 0, ctx->stream, Sk, sb, nbk,
                               trans ? 0 : 1, b + k0, sol + k0, badd != nullptr ? badd + k0 : nullptr, scale,
                               badd != nullptr ? bout + k0 : nullptr, out32 != nullptr ? out32 + k0 : nullptr);
            if (hi == lo) continue;
            auto panel = [&](auto kernel, int outs, int threads) { // outs: of a workgroup
                hipLaunchKernelGGL(kernel, dim3((unsigned)((hi - lo + outs - 1) / outs)), dim3(threads), 0, ctx->stream, R, ld, k0, nbk, lo, hi, sol + k0, b,
                                   work);
            };
            if (trans == lower)
                hi - lo <= kPanelShortUpTo ? panel(panel_update_n_kernel<16>, 16, kPanelWaves * 64) : panel(panel_update_n_kernel<32>, 32, kPanelWaves * 64);
            else
                panel(panel_update_t_kernel, 4, 256);
        }
        if (tc > 1)
            hipLaunchKernelGGL(rows16_to_cols_kernel, grid1(M * tc), dim3(256), 0, ctx->stream, p->xw, half, M, tc, bout, M, badd, scale);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "blocked triangular solve", e);
    return KNM_OK;
}

// S <- mirrored inverses of the sb x sb diagonal blocks of the upper-triangular R (p->T or p->A).  S holds the
// inverses of the 128 x 128 diagonal blocks, which the leaf kernel left there, and zeros; neighbouring inverses are
// merged level by level,  inv([R11 R12; 0 R22]) = [W11, -W11 R12 W22; 0, W22],  with two products for all pairs of
// a level, until the blocks are sb wide; last the upper triangle of every block is copied onto its lower.
int invert_diag_blocks(knm_ctx *ctx, const knm_precond *p, const double *R, double *S)
{
    const int64_t M = p->M, ld = p->ld;
    const int lower = (R == p->A) ? 1 : 0;
    const int sb = p->sb;
    const int64_t nblk = (M + sb - 1) / sb;
    if (launch_merge_inverses(R, ld, lower, M, S, sb, ctx->stream) != hipSuccess)
        return fail(ctx, KNM_HIP_ERROR, "inverse merge launch");
    hipLaunchKernelGGL(mirror_upper_kernel, dim3((unsigned)((sb + 255) / 256), (unsigned)sb, (unsigned)nblk), dim3(256),
                       0, ctx->stream, S, sb);
    if (hipGetLastError() != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "diagonal block inversion launch");
    return KNM_OK;
}

// Workspace of one application of the operator of Eq. 9 on column-major fp64 vectors.
struct LinopWork {
    DevBuf v, w, c, z32, u32, u64;
    int alloc(knm_ctx *ctx, int64_t M, int t)
    {
        int st = v.alloc(ctx, sizeof(double) * M * t);
        if (!st) st = w.alloc(ctx, sizeof(double) * M * t);
        if (!st) st = c.alloc(ctx, sizeof(double) * M * t);
        if (!st) st = z32.alloc(ctx, sizeof(float) * M * t);
        if (!st) st = u32.alloc(ctx, sizeof(float) * M * t);
        if (!st) st = u64.alloc(ctx, sizeof(double) * M * t);
        return st;
    }
};

// The two sweeps of one (X, C, sigma), whatever the storage of the points: W (n x t) = K V and
// U (M x t) = K^T (wgt .* W) (wgt over the rows of X, or null)
struct KernelOps {
    int64_t n = 0, M = 0;
    std::function<int(const float *V, int t, float *W)> v;
    std::function<int(const float *W, const float *wgt, int t, float *U)> t_w;
    // the same with U as fp64 rows (M x t, row-major) that were never rounded to fp32; may be empty
    std::function<int(const float *W, const float *wgt, int t, double *U64)> t_w64;
};

// Operand conversions the split-fp16 engines have clamped so far (waits for the stream).
int read_range_count(knm_ctx *ctx, unsigned int *count)
{
    hipError_t e = hipMemcpyAsync(count, ctx->range_count, sizeof(*count), hipMemcpyDeviceToHost, ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    return e == hipSuccess ? KNM_OK : fail(ctx, KNM_HIP_ERROR, "range counter", e);
}

// A fit runs with the context's cross-term mode unless its first sweep had to clamp operands (points
// outside the range of the split-fp16 engines): then the whole fit runs on the fp32 matrix cores,
// which have no such limits, and the context's mode comes back when the fit returns.
struct CrossTermScope {
    knm_ctx *ctx;
    int saved;
    unsigned int before = 0;
    explicit CrossTermScope(knm_ctx *c) : ctx(c), saved(c->cross_term) {}
    ~CrossTermScope() { ctx->cross_term = saved; }
    int begin() { return read_range_count(ctx, &before); }
    // after the first sweep: true if it must be repeated in the fp32 mode (now selected)
    int check(bool *repeat)
    {
        *repeat = false;
        if (ctx->cross_term != KNM_CROSS_F16X3) return KNM_OK;
        unsigned int now = 0;
        int st = read_range_count(ctx, &now);
        if (st) return st;
        if (now != before) {
            ctx->cross_term = KNM_CROSS_F32;
            *repeat = true;
        }
        return KNM_OK;
    }
};

// cols (M x t, column-major fp64) <- K^T (wgt .* W): T^-T amplifies what the solver is given by the
// conditioning of K_MM, so the result of the column sweep is taken in fp64 where the sweeps offer it
int t_w_cols(knm_ctx *ctx, const KernelOps &ops, const float *W, const float *wgt, int t, float *u32, double *u64,
             double *cols)
{
    if (ops.t_w64) {
        if (t == 1) return ops.t_w64(W, wgt, t, cols); // one column: the same array either way
        int st = ops.t_w64(W, wgt, t, u64);
        if (st) return st;
        hipLaunchKernelGGL(f64_rows_to_cols, grid1(ops.M * t), dim3(256), 0, ctx->stream, u64, ops.M, t, cols, 0);
    } else {
        int st = ops.t_w(W, wgt, t, u32);
        if (st) return st;
        hipLaunchKernelGGL(f32_rows_to_f64_cols, grid1(ops.M * t), dim3(256), 0, ctx->stream, u32, ops.M, t, cols);
    }
    return hipGetLastError() == hipSuccess ? KNM_OK : fail(ctx, KNM_HIP_ERROR, "column sweep result conversion");
}

KernelOps dense_ops(knm_ctx *ctx, const float *X, int64_t n, int d, int64_t ldx, const float *C, int64_t M, int64_t ldc,
                    float sigma)
{
    KernelOps ops;
    ops.n = n;
    ops.M = M;
    ops.v = [=](const float *V, int t, float *W) { return do_knm_v(ctx, X, n, d, ldx, C, M, ldc, sigma, V, t, W); };
    ops.t_w = [=](const float *W, const float *wgt, int t, float *U) {
        return do_knm_t_w(ctx, X, n, d, ldx, C, M, ldc, sigma, W, wgt, t, U);
    };
    ops.t_w64 = [=](const float *W, const float *wgt, int t, double *U64) {
        return do_knm_t_w(ctx, X, n, d, ldx, C, M, ldc, sigma, W, wgt, t, nullptr, U64);
    };
    return ops;
}

// out <- A^-T ( T^-T K^T D K T^-1 A^-1 beta + lambda n A^-1 beta );  beta, out column-major, may not alias;
// D = diag(wgt) over the rows of X, identity if wgt is null
int linop_cols(knm_ctx *ctx, const knm_precond *p, LinopWork &wk, const KernelOps &ops, double lambda,
               const double *beta, int t, double *out, const float *wgt = nullptr)
{
    const int64_t n = ops.n, M = ops.M;
    double *v = wk.v.as<double>(), *w = wk.w.as<double>(), *c = wk.c.as<double>();
    float *z32 = wk.z32.as<float>();
    int st = tri_solve(ctx, p, p->A, p->Adinv, false, beta, v, t); // v = A^-1 beta
    if (!st) st = tri_solve(ctx, p, p->T, p->Tdinv, false, v, w, t, nullptr, 0.0, t == 1 ? z32 : nullptr); // z = T^-1 v
    if (st) return st;
    if (t > 1) hipLaunchKernelGGL(f64_cols_to_f32_rows, grid1(M * t), dim3(256), 0, ctx->stream, w, M, t, z32);
    // c = K_nm^T (K_nm z), the O(n M) step
    st = ensure(ctx, &ctx->w_buf, &ctx->w_bytes, sizeof(float) * (size_t)n * t);
    if (st) return st;
    st = ops.v(z32, t, ctx->w_buf);
    if (st) return st;
    st = t_w_cols(ctx, ops, ctx->w_buf, wgt, t, wk.u32.as<float>(), wk.u64.as<double>(), c);
    if (st) return st;
    st = tri_solve(ctx, p, p->T, p->Tdinv, true, c, w, t, v, lambda * (double)n); // T^-T c + lambda n v
    if (st) return st;
    return tri_solve(ctx, p, p->A, p->Adinv, true, w, out, t); // A^-T (...)
}

} // namespace

extern "C" {

void knm_solver_release(knm_ctx *ctx)
{
    for (int i = 0; ctx && i < 2; ++i)
        if (ctx->fit_ev[i]) {
            (void)hipEventDestroy(ctx->fit_ev[i]);
            ctx->fit_ev[i] = nullptr;
        }
    if (ctx && ctx->aux_stream) {
        (void)hipStreamDestroy(ctx->aux_stream);
        ctx->aux_stream = nullptr;
    }
}

int precond_free(knm_precond *p)
{
    if (!p) return KNM_INVALID_ARG;
    (void)hipSetDevice(p->device);
    for (double *a : {p->buf, p->Tdinv, p->Adinv, p->xw, p->blk}) {
        if (!a) continue;
        if (p->pool) pool_give(p->pool, a);
        else (void)hipFree(a);
    }
    delete p;
    return KNM_OK;
}

// Upper Cholesky factor in place, R^T R = A (upper or lower storage, leading dimension ld): the three-step
// column update of Sec. 4 (block Cholesky paragraph) on block rows of up to 4096.
//   Steps 1 and 2 (factor the diagonal tile, solve the block row against it) are carried out
//   together, left-looking over sub-panels of 512 rows and, inside them, steps of 128 rows: a
//   row group, from its diagonal to the last column, first loses the products with the rows
//   above it (one block product, contraction over the rows already done), then the diagonal
//   block of a step is factorised and inverted by the leaf kernel, then the rest of its rows is
//   multiplied by that inverse (in place: a 128-row tile of the block product reads exactly
//   the columns it writes).
//   Step 3 (trailing update, M^3 / 3 of the flop) is one rank-k launch per block row.
// S (as many sb x sb column-major blocks as cover M) is cleared and receives the inverses of the 128 x 128 diagonal
// blocks at their places; `bad` is a device word that receives the least 1-based index of a failing pivot (all ones: none).
constexpr int64_t kSubPanel = 512;

// events without timing, destroyed with the set
struct EventSet {
    std::vector<hipEvent_t> ev;
    ~EventSet()
    {
        for (hipEvent_t e : ev)
            if (e) (void)hipEventDestroy(e);
    }
    bool create(int64_t count)
    {
        ev.assign((size_t)count, nullptr);
        for (auto &e : ev)
            if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) return false;
        return true;
    }
    hipEvent_t operator[](int64_t i) const { return ev[(size_t)i]; }
};

// second stream of the context (default priority, no implicit ordering with the legacy default
// stream: every dependency is an event), created on first use
static int aux_stream(knm_ctx *ctx, hipStream_t *out)
{
    if (!ctx->aux_stream) {
        hipStream_t s = nullptr;
        hipError_t e = hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
        if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipStreamCreateWithFlags", e);
        ctx->aux_stream = s;
    }
    *out = ctx->aux_stream;
    return KNM_OK;
}

// What building a preconditioner that the caller keeps leaves idle in the pool: up to 4 GiB (all of it at M = 20000), as fits do; the 12 GiB of
// M = 100000 go back to the device.
struct IdleScope {
    knm_ctx *ctx;
    size_t before;
    explicit IdleScope(knm_ctx *c) : ctx(c), before(c ? pool_idle_bytes(c) : 0) {}
    ~IdleScope()
    {
        if (ctx) pool_trim(ctx, std::max(before, (size_t)4 << 30));
    }
};

// Room for updates by residues, from the pool: given back when it goes out of scope, in the order of the context's stream.
struct ResidueRoom {
    knm_ctx *ctx;
    bool ok = false;
    DevBuf img[2], exps[2], bytes[2];
    size_t bytes_size[2] = {0, 0};
    explicit ResidueRoom(knm_ctx *c) : ctx(c) {}
    // Operands of up to n rows over K, in `sets` sets; the sums of an n x n matrix and, with first_rows, of that many rows of it
    // apart.  At most kBytes of either at a time.
    static constexpr size_t kBytes = (size_t)1 << 30;
    void take(int64_t n, int64_t K, int sets, int64_t first_rows)
    {
        ok = true;
        for (int s = 0; s < sets && ok; ++s)
            ok = img[s].alloc_for_speed(ctx, residue_image_bytes(n, K)) && exps[s].alloc_for_speed(ctx, sizeof(int) * (size_t)n);
        // (both storages: strips of `first_rows` x n and n x n entries whichever index is the contiguous one)
        if (first_rows > 0) bytes_size[0] = std::max(residue_bytes(first_rows, n, kBytes / 2), residue_bytes(n, first_rows, kBytes / 2));
        bytes_size[1] = residue_bytes(n, n, kBytes);
        for (int k = 0; k < 2 && ok; ++k) ok = bytes_size[k] == 0 || bytes[k].alloc_for_speed(ctx, bytes_size[k]);
        if (!ok) // (what was found goes back to the device: the card is nearly full)
            for (DevBuf *part : {&img[0], &img[1], &exps[0], &exps[1], &bytes[0], &bytes[1]}) part->drop();
    }
};

// `lower`: the factor and the matrix it replaces are in lower storage (entry (r, c), r <= c, at
// A[c + r ld]); every product below then has its two index roles exchanged.  A block row that straddles the
// diagonal is stored on its own side only, because the other triangle belongs to the other factor.
static int chol_blocked(knm_ctx *ctx, double *A, int64_t ld, int64_t M, bool lower, double *S, int sb,
                        unsigned long long *bad)
{
    TraceRange range(lower ? "knm Cholesky of T D T^T / M + lambda I" : "knm Cholesky of K_MM");
    int64_t b = ((M + 7) / 8 + 255) / 256 * 256;
    if (b > 4096) b = 4096;
    const int64_t nb = (M + b - 1) / b;
    hipError_t e = hipMemsetAsync(bad, 0xff, sizeof(*bad), ctx->stream);
    if (e == hipSuccess) e = hipMemsetAsync(S, 0, sizeof(double) * (size_t)((M + sb - 1) / sb) * sb * sb, ctx->stream);
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipMemsetAsync", e);
    hipStream_t aux = nullptr;
    int st = aux_stream(ctx, &aux);
    if (st) return st;
    // The trailing updates as integer products modulo small numbers (knm_residue.hip) where that is faster and there is room: planes of
    // a block row in two sets in turn, so that those of the next are made while the rest of the update still reads these,
    // and the residues of the sums, of the part on either stream.
    ResidueRoom residues(ctx);
    if (M > b && residue_pays(M - b, b, false)) residues.take(M - b, b, 2, b);
    // on an early return the arrays may go back to the pool, whose blocks are ordered by the context's stream only
    struct AuxJoin {
        hipStream_t s;
        ~AuxJoin()
        {
            if (s) (void)hipStreamSynchronize(s);
        }
    } join{aux};
    EventSet ev_rows, ev_rest;
    if (!ev_rows.create(nb) || !ev_rest.create(nb)) return fail(ctx, KNM_HIP_ERROR, "hipEventCreate");
    std::vector<char> have_rest(nb, 0);
    // entry (r, c) of the matrix, r <= c
    auto at = [&](int64_t r, int64_t c) { return lower ? A + c + (size_t)r * ld : A + r + (size_t)c * ld; };
    // rows [row, row + nr) of the columns from `col` on lose the products with rows [top, top + K)
    // of the same columns: R(row + i, col + j) -= sum_k R(top + k, row + i) R(top + k, col + j).
    // Here col == row: the triangle of the nr x nr block on the diagonal and the rectangle to its right.
    auto update_rows = [&](int64_t top, int64_t K, int64_t row, int64_t nr) -> bool {
        const int64_t ncols = M - row;
        const double *P = at(top, row); // element (top + k, row + x) at P[k + x ld], or P[x + k ld] in lower storage
        return (lower ? launch_gemm_f64(1, ncols, nr, K, -1.0, P, ld, P, ld, 1.0, at(row, row), ld, ctx->stream, 1, 2)
                      : launch_gemm_f64(0, nr, ncols, K, -1.0, P, ld, P, ld, 1.0, at(row, row), ld, ctx->stream, 0, 1)) == hipSuccess;
    };
    for (int64_t k = 0; k < nb; ++k) {
        const int64_t r0 = k * b;
        const int64_t w = (M - r0 < b) ? M - r0 : b;
        for (int64_t S0 = 0; S0 < w; S0 += kSubPanel) {
            // the sub-panel's rows lose the products with the block row's rows above them at once
            // (four tile rows per launch); inside it the 128-row steps only reach back to its top
            const int64_t sw = (w - S0 < kSubPanel) ? w - S0 : kSubPanel;
            const int64_t prow = r0 + S0;
            for (int64_t s0 = 0; s0 < sw; s0 += kLeaf) {
                const int64_t row = prow + s0;
                const int nbk = (int)((sw - s0 < kLeaf) ? sw - s0 : kLeaf);
                const int64_t ncols = M - row;
                const LeafArgs leaf = {at(row, row), ld, nbk, S + (row / sb) * (int64_t)sb * sb + (row % sb) * (int64_t)(sb + 1), // sb is a multiple of 128
                                       (int64_t)sb, row, bad, lower ? 1 : 0};
                double *const W = leaf.W;
                // the rows above that reach into these: of the block row for the first step of a sub-panel, of the sub-panel for the others
                const int64_t top = s0 > 0 ? prow : r0, K = row - top, nr = s0 > 0 ? nbk : sw;
                if (nbk == kLeaf && leaf_hides_update(nr, ncols, K)) {
                    // the diagonal block first, then its factorisation beside the rest
                    const double *P = at(top, row);
                    hipError_t le = lower ? launch_gemm_f64(1, nbk, nbk, K, -1.0, P, ld, P, ld, 1.0, leaf.A, ld, ctx->stream, 1, 2)
                                          : launch_gemm_f64(0, nbk, nbk, K, -1.0, P, ld, P, ld, 1.0, leaf.A, ld, ctx->stream, 0, 1);
                    if (le == hipSuccess) le = launch_leaf_beside_update(leaf, lower ? ncols : nr, lower ? nr : ncols, K, P, ctx->stream);
                    if (le != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "block row update launch");
                } else {
                    if (K > 0 && !update_rows(top, K, row, nr)) return fail(ctx, KNM_HIP_ERROR, "block row update launch");
                    hipLaunchKernelGGL(potrf_trtri_leaf_kernel, dim3(1), dim3(kLeafThreads), 0, ctx->stream, leaf);
                }
                if (ncols > nbk) {
                    // the rest of the rows times the inverse: R(row + i, c) <- sum_k W(k, i) R(row + k, c)
                    double *right = at(row, row + nbk);
                    const hipError_t le =
                        lower ? launch_gemm_f64(1, ncols - nbk, nbk, nbk, 1.0, right, ld, W, sb, 0.0, right, ld, ctx->stream, 0, 0, true)
                              : launch_gemm_f64(0, nbk, ncols - nbk, nbk, 1.0, W, sb, right, ld, 0.0, right, ld, ctx->stream, 0, 0, true);
                    if (le != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "block row solve launch");
                }
            }
        }
        const int64_t rest = M - r0 - w;
        if (rest == 0) break;
        // Step 3 with one block row of look-ahead.  The part of the trailing matrix that the next
        // block row needs (its own rows) is updated on the main stream, which then goes on to
        // steps 1 and 2 of that block row; the remainder (most of the flop) runs on the second
        // stream meanwhile and fills the chip, which those short dependent launches cannot.
        const int64_t w2 = (rest < b) ? rest : b;
        const int64_t c0 = r0 + w;                 // first trailing row and column
        const double *Akr2 = at(r0, c0 + w2);      // block row to the right of the columns of the next one
        const int form = lower ? 1 : 0, tc = lower ? 1 : 0;
        const bool by_residues = residues.ok && residue_pays(rest, w, false);
        ResidueUpdate up = {};
        if (by_residues) {
            const int set = (int)(k & 1);
            up.img_u = up.img_v = residues.img[set].p;
            up.exp_u = up.exp_v = residues.exps[set].as<int>();
            up.n = rest;
            up.K = w;
            up.lower = lower ? 1 : 0;
            up.alpha = -1.0;
            up.beta = 1.0;
            up.C = at(c0, c0);
            up.ldc = ld;
            if (launch_residue_image(form, rest, w, at(r0, c0), ld, nullptr, 0, 0, residues.exps[set].as<int>(), residues.img[set].p,
                                     ctx->stream) != hipSuccess)
                return fail(ctx, KNM_HIP_ERROR, "trailing update launch");
        }
        // rows [i0, i1) of the trailing matrix from column j0 on lose their part of the update
        auto update_by_residues = [&](int64_t i0, int64_t i1, int64_t j0, int which, hipStream_t stream) -> bool {
            ResidueUpdate q = up;
            (lower ? q.v0 : q.u0) = i0;
            (lower ? q.v1 : q.u1) = i1;
            (lower ? q.u0 : q.v0) = j0;
            (lower ? q.u1 : q.v1) = rest;
            q.bytes = residues.bytes[which].p;
            q.bytes_size = residues.bytes_size[which];
            return launch_residue_update(q, stream) == hipSuccess;
        };
        if (hipEventRecord(ev_rows[k], ctx->stream) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipEventRecord");
        if (k > 0 && have_rest[k - 1] && hipStreamWaitEvent(ctx->stream, ev_rest[k - 1], 0) != hipSuccess)
            return fail(ctx, KNM_HIP_ERROR, "hipStreamWaitEvent");
        if (!(by_residues ? update_by_residues(0, w2, 0, 0, ctx->stream) : update_rows(r0, w, c0, w2)))
            return fail(ctx, KNM_HIP_ERROR, "trailing update launch");
        if (rest > w2) {
            if (hipStreamWaitEvent(aux, ev_rows[k], 0) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipStreamWaitEvent");
            if (by_residues) {
                if (!update_by_residues(w2, rest, w2, 1, aux)) return fail(ctx, KNM_HIP_ERROR, "trailing update launch");
            } else if (launch_rank_k_upper(form, rest - w2, w, -1.0, Akr2, ld, nullptr, 0, 1.0, 0.0, at(c0 + w2, c0 + w2), ld, aux,
                                    tc) != hipSuccess)
                return fail(ctx, KNM_HIP_ERROR, "trailing update launch");
            if (hipEventRecord(ev_rest[k], aux) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipEventRecord");
            have_rest[k] = 1;
        }
    }
    // the second stream's last update (its stream order makes it the last of all) before anything else
    for (int64_t k = nb - 1; k >= 0; --k)
        if (have_rest[k]) {
            if (hipStreamWaitEvent(ctx->stream, ev_rest[k], 0) != hipSuccess)
                return fail(ctx, KNM_HIP_ERROR, "hipStreamWaitEvent");
            break;
        }
    join.s = nullptr; // ordered before whatever follows on the context's stream
    e = hipGetLastError();
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "factorisation", e);
    return KNM_OK;
}

// The words of failing pivots of `count` factorisations (waits for the stream); pivot[k] = 0 for none.
static int read_bad_pivots(knm_ctx *ctx, const unsigned long long *bad, int count, int64_t *pivot)
{
    unsigned long long got[2];
    hipError_t e = hipMemcpyAsync(got, bad, sizeof(*got) * count, hipMemcpyDeviceToHost, ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e == hipSuccess) e = hipGetLastError();
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "factorisation", e);
    for (int k = 0; k < count; ++k) pivot[k] = (got[k] == ~0ull) ? 0 : (int64_t)got[k];
    return KNM_OK;
}

// The update of launch_rank_k_upper (there: form_nt, w, tri; lower: entry (i, j), i <= j, at C[j + i ldc]; tri needs K = n) by residues: 1, or 0 where there is
// no room.  The contraction is taken in slabs of `depth` (0: whose planes fill at most 2 GiB), the last first: with tri its sums reach every entry.  The
// weights go to the two sides as their roots, so that a product of entries is scaled as the sum it is part of; their signs go to one
// side, whose planes are made only where there are any.
static int rank_k_by_residues(knm_ctx *ctx, int form_nt, int lower, int64_t n, int64_t K, int64_t depth, double alpha, const double *A, int64_t lda,
                              const double *w, int tri, double beta, double shift, double *C, int64_t ldc)
{
    const int sides = w != nullptr ? 2 : 1;
    if (depth <= 0) {
        const int64_t per_k = (int64_t)(residue_image_bytes(n, 64) / 64) * sides;
        depth = ((int64_t)2 << 30) / per_k;
        if (depth < 1024) depth = 1024;
        if (depth > residue_max_k()) depth = residue_max_k();
        const int64_t slabs = (K + depth - 1) / depth;
        depth = ((K + slabs - 1) / slabs + 63) / 64 * 64;
    }
    ResidueRoom room(ctx);
    room.take(n, depth < K ? depth : K, sides, 0);
    DevBuf roots, sign;
    if (!room.ok || (w != nullptr && !(roots.alloc_for_speed(ctx, sizeof(double) * 2 * (size_t)K) && sign.alloc_for_speed(ctx, sizeof(int)))))
        return 0;
    double *root[2] = {nullptr, nullptr};
    if (w != nullptr) {
        root[0] = roots.as<double>();
        root[1] = root[0] + K;
        if (launch_signed_root(w, K, root[0], root[1], sign.as<int>(), ctx->stream) != hipSuccess)
            return fail(ctx, KNM_HIP_ERROR, "update by residues");
    }
    int *const exps = room.exps[0].as<int>();
    for (int64_t k1 = K; k1 > 0;) {
        const int64_t k0 = (k1 - 1) / depth * depth, rows = tri ? k1 : n;
        hipError_t e = hipSuccess;
        for (int s = 0; s < sides && e == hipSuccess; ++s)
            e = launch_residue_image(form_nt, rows, k1 - k0, A + (form_nt ? k0 * lda : k0), lda, root[s] ? root[s] + k0 : nullptr, tri, k0, exps,
                                     room.img[s].p, ctx->stream, s == 1 ? sign.as<int>() : nullptr);
        ResidueUpdate up = {};
        up.img_u = room.img[0].p;
        up.img_v = room.img[sides - 1].p;
        up.differ = w != nullptr ? sign.as<int>() : nullptr;
        up.exp_u = up.exp_v = exps;
        up.n = rows;
        up.K = k1 - k0;
        up.u1 = up.v1 = rows;
        up.lower = lower;
        up.tri = tri;
        up.k0 = k0;
        up.alpha = alpha;
        up.beta = k1 == K ? beta : 1.0;
        up.shift = k1 == K ? shift : 0.0;
        up.C = C;
        up.ldc = ldc;
        up.bytes = room.bytes[1].p;
        up.bytes_size = room.bytes_size[1];
        if (e == hipSuccess) e = launch_residue_update(up, ctx->stream);
        if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "update by residues", e);
        k1 = k0;
    }
    return 1;
}

// A <- upper Cholesky factor of T D T^T / M + lambda I, D = diag(dw) (identity if dw is null), and
// the inverses of its diagonal blocks.  T is upper triangular, so entry (i, j) of the product
// only sums over k >= max(i, j): M^3 / 3 flop instead of the M^3 of a dense rank-M update,
// in one launch of the rank-k kernel, which skips the vanishing part tile by tile.  The product is
// written mirrored, into the lower storage of A beside T, and factorised there in place.
// Enqueued only; *bad_dev receives what chol_blocked leaves in its word.
static int build_second_factor(knm_ctx *ctx, knm_precond *p, double lambda, const double *dw, unsigned long long *bad_dev)
{
    const int64_t M = p->M;
    {
        TraceRange range("knm triangular product T D T^T");
        const int by_residues = !residue_pays(M, M, true) ? 0
                                                          : rank_k_by_residues(ctx, 1, 1, M, M, 0, 1.0 / (double)M, p->T, p->ld, dw, 1, 0.0, lambda, p->A, p->ld);
        if (by_residues < 0) return by_residues;
        if (by_residues == 0 && launch_rank_k_upper(1, M, M, 1.0 / (double)M, p->T, p->ld, dw, 1, 0.0, lambda, p->A, p->ld, ctx->stream, 1) !=
            hipSuccess)
            return fail(ctx, KNM_HIP_ERROR, "triangular product launch");
    }
    int st = chol_blocked(ctx, p->A, p->ld, M, true, p->Adinv, p->sb, bad_dev);
    if (!st) st = invert_diag_blocks(ctx, p, p->A, p->Adinv);
    if (!st) p->lambda = lambda;
    return st;
}
static const char *const kSecondNotPd = "T D T^T / M + lambda I is not positive definite";

// fill_kmm(K, ldk) writes the upper triangle of K_MM + jitter I (column-major, leading dimension ldk)
// (pooled: the arrays come from the context's pool, for a preconditioner that does not outlive the call)
static int precond_build_from(knm_ctx *ctx, int64_t M, const std::function<int(double *, int64_t)> &fill_kmm, double lambda,
                              double jitter, bool second_factor, bool pooled, knm_precond **out, int64_t *bad_pivot_or_null)
{
    if (!ctx) return KNM_INVALID_ARG;
    if (!out) return fail(ctx, KNM_INVALID_ARG, "null output");
    *out = nullptr;
    if (bad_pivot_or_null) *bad_pivot_or_null = 0;
    if (M <= 0 || !(lambda >= 0.0) || !(jitter >= 0.0)) return fail(ctx, KNM_INVALID_ARG, "bad preconditioner argument");
    if (M > 2000000000LL / 1) return fail(ctx, KNM_UNSUPPORTED, "M too large");
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipSetDevice");
    int st = KNM_OK;

    knm_precond *p = new (std::nothrow) knm_precond();
    if (!p) return fail(ctx, KNM_ALLOC, "host allocation");
    p->device = ctx->device;
    p->M = M;
    p->lambda = lambda;
    p->jitter = jitter;
    p->ld = M + 2 + (M & 1); // even: every column of either factor starts 16-byte aligned
    p->pool = pooled ? ctx : nullptr;
    p->sb = solve_block_width(M);
    const int64_t nblk = (M + p->sb - 1) / p->sb;
    auto take = [&](double **a, int64_t count) {
        void *ptr = nullptr;
        const size_t bytes = sizeof(double) * (size_t)count;
        const hipError_t err = pooled ? pool_take(ctx, bytes, &ptr) : device_alloc(ctx, bytes, &ptr);
        if (err == hipSuccess) *a = static_cast<double *>(ptr);
        return err;
    };
    hipError_t e = take(&p->buf, p->ld * M);
    p->T = p->buf;
    p->A = p->buf ? p->buf + 2 : nullptr;
    if (e == hipSuccess) e = take(&p->Tdinv, nblk * p->sb * p->sb);
    if (e == hipSuccess) e = take(&p->Adinv, nblk * p->sb * p->sb);
    if (e == hipSuccess) e = take(&p->xw, 4 * M * kSolveCols);
    if (e == hipSuccess && M >= kProductSolveMinM) e = take(&p->blk, (int64_t)p->sb * p->sb);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        precond_free(p);
        return fail(ctx, KNM_ALLOC, "hipMalloc(preconditioner)", e);
    }
    auto bail = [&](int status, const char *what) {
        precond_free(p);
        return fail(ctx, status, what);
    };

    st = fill_kmm(p->T, p->ld);
    if (st) {
        precond_free(p);
        return st;
    }

    // both factors are enqueued before the host asks how the first one went (a failed pivot leaves numbers, not faults)
    DevBuf badbuf;
    if (badbuf.alloc(ctx, 2 * sizeof(unsigned long long))) return bail(KNM_ALLOC, "hipMalloc");
    unsigned long long *bad = badbuf.as<unsigned long long>();
    st = chol_blocked(ctx, p->T, p->ld, M, false, p->Tdinv, p->sb, bad);
    if (!st) st = invert_diag_blocks(ctx, p, p->T, p->Tdinv);
    if (!st && second_factor) st = build_second_factor(ctx, p, lambda, nullptr, bad + 1);
    int64_t pivot[2] = {0, 0};
    if (!st) st = read_bad_pivots(ctx, bad, second_factor ? 2 : 1, pivot);
    if (st) {
        precond_free(p);
        return st;
    }
    if (pivot[0] != 0 || pivot[1] != 0) {
        if (bad_pivot_or_null) *bad_pivot_or_null = pivot[0] != 0 ? pivot[0] : -pivot[1];
        return bail(KNM_NOT_PD, pivot[0] != 0 ? "K_MM + jitter I is not positive definite" : kSecondNotPd);
    }
    *out = p;
    return KNM_OK;
}

static int precond_build_impl(knm_ctx *ctx, const float *C, int64_t M, int d, int64_t ldc, float sigma, double lambda,
                              double jitter, bool second_factor, bool pooled, knm_precond **out, int64_t *bad_pivot_or_null)
{
    if (!ctx) return KNM_INVALID_ARG;
    if (!C || M <= 0 || d <= 0 || ldc < d || !(sigma > 0.0f))
        return fail(ctx, KNM_INVALID_ARG, "bad preconditioner argument");
    auto fill = [=](double *K, int64_t ldk) {
        const dim3 tb(256);
        const dim3 tg((unsigned)((M + kKmmTile - 1) / kKmmTile), (unsigned)((M + kKmmTile - 1) / kKmmTile));
        const int kind = ctx->kernel_kind;
        const double scale = kind == KNM_KERNEL_GAUSSIAN   ? 1.0 / (2.0 * (double)sigma * (double)sigma)
                             : kind == KNM_KERNEL_MATERN32 ? sqrt(3.0) / (double)sigma
                             : kind == KNM_KERNEL_MATERN52 ? sqrt(5.0) / (double)sigma
                                                           : 1.0 / (double)sigma;
        hipLaunchKernelGGL(kmm_kernel, tg, tb, 0, ctx->stream, C, M, d, ldc, kind, scale, jitter, K, ldk);
        return hipGetLastError() == hipSuccess ? KNM_OK : fail(ctx, KNM_HIP_ERROR, "kmm_kernel launch");
    };
    return precond_build_from(ctx, M, fill, lambda, jitter, second_factor, pooled, out, bad_pivot_or_null);
}

int precond_build(knm_ctx *ctx, const float *C, int64_t M, int d, int64_t ldc, float sigma, double lambda,
                  double jitter, knm_precond **out, int64_t *bad_pivot_or_null)
{
    const IdleScope idle(ctx);
    return precond_build_impl(ctx, C, M, d, ldc, sigma, lambda, jitter, true, false, out, bad_pivot_or_null);
}

static int precond_build_csr_impl(knm_ctx *ctx, const int64_t *c_indptr, const int64_t *c_indices, const float *c_values, int64_t M,
                      int64_t d, float sigma, double lambda, double jitter, bool second_factor, bool pooled,
                      knm_precond **out, int64_t *bad_pivot_or_null)
{
    if (!ctx) return KNM_INVALID_ARG;
    if (!c_indptr || M <= 0 || d <= 0 || d >= 0x7fffffffLL || !(sigma > 0.0f))
        return fail(ctx, KNM_INVALID_ARG, "bad preconditioner argument");
    auto fill = [=](double *K, int64_t ldk) {
        return sparse_kmm(ctx, c_indptr, c_indices, c_values, M, d, sigma, jitter, K, ldk);
    };
    return precond_build_from(ctx, M, fill, lambda, jitter, second_factor, pooled, out, bad_pivot_or_null);
}

int precond_build_csr(knm_ctx *ctx, const int64_t *c_indptr, const int64_t *c_indices, const float *c_values, int64_t M,
                      int64_t d, float sigma, double lambda, double jitter, knm_precond **out,
                      int64_t *bad_pivot_or_null)
{
    const IdleScope idle(ctx);
    return precond_build_csr_impl(ctx, c_indptr, c_indices, c_values, M, d, sigma, lambda, jitter, true, false, out,
                                  bad_pivot_or_null);
}

int precond_get_factors(knm_ctx *ctx, const knm_precond *p, double *T_host, double *A_host)
{
    if (!ctx || !p) return KNM_INVALID_ARG;
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipSetDevice");
    const int64_t M = p->M;
    std::vector<double> tmp((size_t)M * M);
    const double *src[2] = {p->T, p->A};
    double *dst[2] = {T_host, A_host};
    for (int k = 0; k < 2; ++k) {
        if (!dst[k]) continue;
        hipError_t e = hipStreamSynchronize(ctx->stream);
        if (e == hipSuccess)
            e = hipMemcpy2D(tmp.data(), sizeof(double) * M, src[k], sizeof(double) * p->ld, sizeof(double) * M, (size_t)M,
                            hipMemcpyDeviceToHost);
        if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipMemcpy(factor)", e);
        // T: upper storage, entry (i, j) at i + j M of the copy; A: lower storage, at j + i M
        for (int64_t i = 0; i < M; ++i)
            for (int64_t j = 0; j < M; ++j) dst[k][i * M + j] = (j >= i) ? (k == 0 ? tmp[i + j * M] : tmp[j + i * M]) : 0.0;
    }
    return KNM_OK;
}

int precond_get_block(knm_ctx *ctx, const knm_precond *p, int second, int64_t row0, int64_t col0, int64_t rows,
                      int64_t cols, double *out_host)
{
    if (!ctx) return KNM_INVALID_ARG;
    if (!p || !out_host || row0 < 0 || col0 < 0 || rows <= 0 || cols <= 0 || row0 + rows > p->M || col0 + cols > p->M)
        return fail(ctx, KNM_INVALID_ARG, "bad factor block");
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipSetDevice");
    // gathered on the device (a row of an upper-storage factor is strided in memory), then one copy
    DevBuf tmp;
    int st = tmp.alloc(ctx, sizeof(double) * (size_t)rows * (size_t)cols);
    if (st) return st;
    hipLaunchKernelGGL(gather_block_kernel, grid1(rows * cols), dim3(256), 0, ctx->stream, second ? p->A : p->T, p->ld,
                       second ? 1 : 0, row0, col0, rows, cols, tmp.as<double>());
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e == hipSuccess) e = hipMemcpy(out_host, tmp.p, sizeof(double) * (size_t)rows * (size_t)cols, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "factor block copy", e);
    return KNM_OK;
}

int falkon_linop_weighted(knm_ctx *ctx, const knm_precond *p, const float *X, int64_t n, int d, int64_t ldx,
                          const float *C, int64_t M, int64_t ldc, float sigma, double lambda, const float *dw_or_null,
                          const double *beta, int t, double *out)
{
    if (!ctx) return KNM_INVALID_ARG;
    if (!p || !X || !C || !beta || !out || n <= 0 || M <= 0 || d <= 0 || t <= 0 || ldx < d || ldc < d ||
        !(sigma > 0.0f) || p->M != M)
        return fail(ctx, KNM_INVALID_ARG, "bad linop argument");
    if (d > knm_max_d() || t > knm_max_t()) return fail(ctx, KNM_UNSUPPORTED, "d or t above compiled maximum");
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipSetDevice");
    int st = KNM_OK;
    LinopWork wk;
    DevBuf bc, oc;
    st = wk.alloc(ctx, M, t);
    if (!st) st = bc.alloc(ctx, sizeof(double) * M * t);
    if (!st) st = oc.alloc(ctx, sizeof(double) * M * t);
    if (st) return st;
    hipLaunchKernelGGL(f64_rows_to_cols, grid1(M * t), dim3(256), 0, ctx->stream, beta, M, t, bc.as<double>(), 0);
    SweepShare share(ctx, X, n, ldx, C, M, ldc, d, sigma, t, false);
    const ShareScope scope(share);
    st = linop_cols(ctx, p, wk, dense_ops(ctx, X, n, d, ldx, C, M, ldc, sigma), lambda, bc.as<double>(), t, oc.as<double>(),
                    dw_or_null);
    if (st) return st;
    hipLaunchKernelGGL(f64_rows_to_cols, grid1(M * t), dim3(256), 0, ctx->stream, oc.as<double>(), M, t, out, 1);
    hipError_t e = hipStreamSynchronize(ctx->stream); // temporaries are freed on return
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "falkon_linop", e);
    return KNM_OK;
}

int falkon_linop(knm_ctx *ctx, const knm_precond *p, const float *X, int64_t n, int d, int64_t ldx, const float *C,
                 int64_t M, int64_t ldc, float sigma, double lambda, const double *beta, int t, double *out)
{
    return falkon_linop_weighted(ctx, p, X, n, d, ldx, C, M, ldc, sigma, lambda, nullptr, beta, t, out);
}

int precond_rank_k_update(knm_ctx *ctx, int form_nt, int64_t n, int64_t k, double alpha, const double *A, int64_t lda,
                          const double *w_or_null, int triangular, double beta, double shift, double *C, int64_t ldc)
{
    if (!ctx) return KNM_INVALID_ARG;
    if (n < 0 || k < 0 || !C || ldc < (n > 1 ? n : 1) || (n > 0 && k > 0 && !A))
        return fail(ctx, KNM_INVALID_ARG, "bad rank-k update argument");
    if (n > 0 && k > 0 && lda < (form_nt ? n : k)) return fail(ctx, KNM_INVALID_ARG, "leading dimension too small");
    if (triangular && !form_nt) return fail(ctx, KNM_INVALID_ARG, "triangular operand needs the row-contiguous form");
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipSetDevice");
    hipError_t e = launch_rank_k_upper(form_nt, n, k, alpha, A, lda, w_or_null, triangular, beta, shift, C, ldc,
                                       ctx->stream);
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "rank-k update launch", e);
    return KNM_OK;
}

int precond_residue_update(knm_ctx *ctx, int form_nt, int lower, int64_t n, int64_t k, int64_t slab, double alpha, const double *A, int64_t lda,
                           const double *w_or_null, int triangular, double beta, double shift, double *C, int64_t ldc)
{
    if (!ctx) return KNM_INVALID_ARG;
    if (n <= 0 || k <= 0 || slab < 0 || !A || !C || ldc < n || lda < (form_nt ? n : k)) return fail(ctx, KNM_INVALID_ARG, "bad rank-k update argument");
    if (slab % 64 != 0 || slab > residue_max_k()) return fail(ctx, KNM_INVALID_ARG, "slabs are multiples of 64 up to 65536");
    if (triangular && (!form_nt || k != n)) return fail(ctx, KNM_INVALID_ARG, "triangular operand needs the row-contiguous form and k = n");
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipSetDevice");
    const int done = rank_k_by_residues(ctx, form_nt, lower, n, k, slab, alpha, A, lda, w_or_null, triangular, beta, shift, C, ldc);
    return done < 0 ? done : done == 0 ? fail(ctx, KNM_ALLOC, "no room for an update by residues") : KNM_OK;
}

int precond_block_product(knm_ctx *ctx, int a_nt, int64_t ni, int64_t nj, int64_t k, double alpha, const double *A,
                          int64_t lda, const double *B, int64_t ldb, double beta, double *C, int64_t ldc)
{
    if (!ctx) return KNM_INVALID_ARG;
    if (ni < 0 || nj < 0 || k < 0 || !C || ldc < (ni > 1 ? ni : 1) || (ni > 0 && nj > 0 && k > 0 && (!A || !B)))
        return fail(ctx, KNM_INVALID_ARG, "bad block product argument");
    if (ni > 0 && nj > 0 && k > 0 && (lda < (a_nt ? ni : k) || ldb < k))
        return fail(ctx, KNM_INVALID_ARG, "leading dimension too small");
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipSetDevice");
    hipError_t e = launch_gemm_f64(a_nt, ni, nj, k, alpha, A, lda, B, ldb, beta, C, ldc, ctx->stream);
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "block product launch", e);
    return KNM_OK;
}

int precond_solve(knm_ctx *ctx, const knm_precond *p, int transpose, const double *b, int t, double *out)
{
    if (!ctx) return KNM_INVALID_ARG;
    if (!p || !b || !out || t <= 0 || t > knm_max_t()) return fail(ctx, KNM_INVALID_ARG, "bad solve argument");
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipSetDevice");
    const int64_t M = p->M;
    DevBuf bc, wc;
    int st = bc.alloc(ctx, sizeof(double) * M * t);
    if (!st) st = wc.alloc(ctx, sizeof(double) * M * t);
    if (st) return st;
    double *v = bc.as<double>(), *w = wc.as<double>();
    hipLaunchKernelGGL(f64_rows_to_cols, grid1(M * t), dim3(256), 0, ctx->stream, b, M, t, v, 0);
    if (transpose) {
        st = tri_solve(ctx, p, p->T, p->Tdinv, true, v, w, t);
        if (!st) st = tri_solve(ctx, p, p->A, p->Adinv, true, w, v, t);
    } else {
        st = tri_solve(ctx, p, p->A, p->Adinv, false, v, w, t);
        if (!st) st = tri_solve(ctx, p, p->T, p->Tdinv, false, w, v, t);
    }
    if (st) return st;
    hipLaunchKernelGGL(f64_rows_to_cols, grid1(M * t), dim3(256), 0, ctx->stream, v, M, t, out, 1);
    hipError_t e = hipStreamSynchronize(ctx->stream); // the temporary is freed on return
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "precond_solve", e);
    return KNM_OK;
}

int precond_reweight(knm_ctx *ctx, knm_precond *p, double lambda, const double *dw_or_null, int64_t *bad_pivot_or_null)
{
    if (!ctx) return KNM_INVALID_ARG;
    if (bad_pivot_or_null) *bad_pivot_or_null = 0;
    if (!p || !(lambda >= 0.0)) return fail(ctx, KNM_INVALID_ARG, "bad preconditioner argument");
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipSetDevice");
    int st = KNM_OK;
    const IdleScope idle(ctx);
    DevBuf badbuf;
    st = badbuf.alloc(ctx, sizeof(unsigned long long));
    if (st) return st;
    int64_t pivot = 0;
    st = build_second_factor(ctx, p, lambda, dw_or_null, badbuf.as<unsigned long long>());
    if (!st) st = read_bad_pivots(ctx, badbuf.as<unsigned long long>(), 1, &pivot);
    if (bad_pivot_or_null) *bad_pivot_or_null = -pivot;
    if (!st && pivot != 0) st = fail(ctx, KNM_NOT_PD, kSecondNotPd);
    return st;
}

// Alg. 1 from the right-hand side on, with the preconditioner built: exactly `iters` steps of
// preconditioned CG on the operator of Eq. 9, then alpha = T^-1 A^-1 beta.  Takes ownership of p.
static int fit_core(knm_ctx *ctx, const KernelOps &ops, knm_precond *p, const float *Y, int t, double lambda, int iters,
                    float *alpha, double *resid_norms_or_null, std::chrono::steady_clock::time_point t_start)
{
    using clk = std::chrono::steady_clock;
    auto secs = [](clk::time_point a, clk::time_point b) { return std::chrono::duration<double>(b - a).count(); };
    const clk::time_point t_precond = clk::now();
    struct Guard {
        knm_precond *p;
        ~Guard() { precond_free(p); }
    } guard{p};
    const int64_t M = ops.M;
    int st = KNM_OK;

    const int64_t len = M * t;
    const int blocks = red_blocks(M);
    const dim3 vgrid((unsigned)blocks, (unsigned)t), vblock(256);
    LinopWork wk;
    DevBuf beta, r, pv, q, scal;
    st = wk.alloc(ctx, M, t);
    if (!st) st = beta.alloc(ctx, sizeof(double) * len);
    if (!st) st = r.alloc(ctx, sizeof(double) * len);
    if (!st) st = pv.alloc(ctx, sizeof(double) * len);
    if (!st) st = q.alloc(ctx, sizeof(double) * len);
    // r . r of every iteration and column, then the partials of p . q and r . r
    if (!st) st = scal.alloc(ctx, sizeof(double) * ((size_t)(iters + 1) * t + 2 * (size_t)blocks * t));
    for (int i = 0; !st && i < 2; ++i)
        if (!ctx->fit_ev[i] && hipEventCreate(&ctx->fit_ev[i]) != hipSuccess) st = fail(ctx, KNM_HIP_ERROR, "hipEventCreate");
    if (st) return st;
    double *db = beta.as<double>(), *dr = r.as<double>(), *dp = pv.as<double>(), *dq = q.as<double>();
    double *rho = scal.as<double>(), *part_pq = rho + (size_t)(iters + 1) * t, *part_rr = part_pq + (size_t)blocks * t;

    // rhs = A^-T T^-T K_nm^T Y
    CrossTermScope cross(ctx);
    st = cross.begin();
    if (st) return st;
    st = t_w_cols(ctx, ops, Y, nullptr, t, wk.u32.as<float>(), wk.u64.as<double>(), wk.c.as<double>());
    if (st) return st;
    bool repeat = false;
    st = cross.check(&repeat);
    if (!st && repeat) st = t_w_cols(ctx, ops, Y, nullptr, t, wk.u32.as<float>(), wk.u64.as<double>(), wk.c.as<double>());
    if (st) return st;
    st = tri_solve(ctx, p, p->T, p->Tdinv, true, wk.c.as<double>(), wk.w.as<double>(), t);
    if (!st) st = tri_solve(ctx, p, p->A, p->Adinv, true, wk.w.as<double>(), dr, t);
    if (st) return st;
    hipError_t e = hipMemsetAsync(db, 0, sizeof(double) * len, ctx->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(dp, dr, sizeof(double) * len, hipMemcpyDeviceToDevice, ctx->stream);
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "CG initialisation", e);
    hipLaunchKernelGGL(dot_partial_kernel, vgrid, vblock, 0, ctx->stream, dr, dr, M, part_rr);
    hipLaunchKernelGGL(dot_finish_kernel, dim3((unsigned)t), dim3(64), 0, ctx->stream, part_rr, blocks, 1.0, rho);
    (void)hipEventRecord(ctx->fit_ev[0], ctx->stream);
    for (int it = 0; it < iters; ++it) {
        TraceRange range("knm CG iteration");
        st = linop_cols(ctx, p, wk, ops, lambda, dp, t, dq);
        if (st) return st;
        const double *now = rho + (size_t)it * t;
        launch_cg_update(ctx->stream, M, t, now, rho + (size_t)(it + 1) * t, dp, dq, db, dr, part_pq, part_rr);
    }
    // alpha = T^-1 A^-1 beta
    st = tri_solve(ctx, p, p->A, p->Adinv, false, db, wk.v.as<double>(), t);
    if (!st) st = tri_solve(ctx, p, p->T, p->Tdinv, false, wk.v.as<double>(), wk.w.as<double>(), t, nullptr, 0.0, t == 1 ? alpha : nullptr);
    if (st) return st;
    if (t > 1) hipLaunchKernelGGL(f64_cols_to_f32_rows, grid1(len), dim3(256), 0, ctx->stream, wk.w.as<double>(), M, t, alpha);
    (void)hipEventRecord(ctx->fit_ev[1], ctx->stream);
    if (resid_norms_or_null)
        e = hipMemcpyAsync(resid_norms_or_null, rho, sizeof(double) * (size_t)(iters + 1) * t, hipMemcpyDeviceToHost, ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream); // the caller's arrays are written, the temporaries done with
    if (e == hipSuccess) e = hipGetLastError();
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "falkon_fit", e);
    if (resid_norms_or_null)
        for (int64_t i = 0; i < (int64_t)(iters + 1) * t; ++i) resid_norms_or_null[i] = std::sqrt(resid_norms_or_null[i]);
    const clk::time_point t_end = clk::now();
    // the iterations run asynchronously: their time is the device's, the right-hand side has what is left
    float iter_ms = 0.0f;
    (void)hipEventElapsedTime(&iter_ms, ctx->fit_ev[0], ctx->fit_ev[1]);
    const double after = secs(t_precond, t_end), its = 1.0e-3 * (double)iter_ms < after ? 1.0e-3 * (double)iter_ms : after;
    ctx->fit_seconds[0] = secs(t_start, t_precond);
    ctx->fit_seconds[1] = after - its;
    ctx->fit_seconds[2] = its;
    ctx->fit_seconds[3] = 0.0;
    return KNM_OK;
}

int falkon_fit(knm_ctx *ctx, const float *X, int64_t n, int d, int64_t ldx, const float *Y, int t, const float *C,
               int64_t M, int64_t ldc, float sigma, double lambda, double jitter, int iters, float *alpha,
               double *resid_norms_or_null)
{
    if (!ctx) return KNM_INVALID_ARG;
    if (!X || !Y || !C || !alpha || n <= 0 || M <= 0 || d <= 0 || t <= 0 || iters <= 0 || ldx < d || ldc < d ||
        !(sigma > 0.0f) || !(lambda >= 0.0) || !(jitter >= 0.0))
        return fail(ctx, KNM_INVALID_ARG, "bad fit argument");
    if (d > knm_max_d() || t > knm_max_t()) return fail(ctx, KNM_UNSUPPORTED, "d or t above compiled maximum");
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipSetDevice");
    const std::chrono::steady_clock::time_point t_start = std::chrono::steady_clock::now();
    knm_precond *p = nullptr;
    int st = precond_build_impl(ctx, C, M, d, ldc, sigma, lambda, jitter, true, true, &p, nullptr); // synchronises
    if (st) return st;
    SweepShare share(ctx, X, n, ldx, C, M, ldc, d, sigma, t, true);
    share.uses = 2 * iters + 1;
    const ShareScope scope(share);
    return fit_core(ctx, dense_ops(ctx, X, n, d, ldx, C, M, ldc, sigma), p, Y, t, lambda, iters, alpha,
                    resid_norms_or_null, t_start);
}

int falkon_fit_csr(knm_ctx *ctx, const int64_t *x_indptr, const int64_t *x_indices, const float *x_values, int64_t n,
                   const float *Y, int t, const int64_t *c_indptr, const int64_t *c_indices, const float *c_values,
                   int64_t M, int64_t d, float sigma, double lambda, double jitter, int iters, float *alpha,
                   double *resid_norms_or_null)
{
    if (!ctx) return KNM_INVALID_ARG;
    if (!x_indptr || !c_indptr || !Y || !alpha || n <= 0 || M <= 0 || d <= 0 || t <= 0 || iters <= 0 ||
        !(sigma > 0.0f) || !(lambda >= 0.0) || !(jitter >= 0.0))
        return fail(ctx, KNM_INVALID_ARG, "bad fit argument");
    if (d >= 0x7fffffffLL || M >= 0x7fffffffLL || t > knm_max_t())
        return fail(ctx, KNM_UNSUPPORTED, "d, M or t above the supported maximum");
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipSetDevice");
    const std::chrono::steady_clock::time_point t_start = std::chrono::steady_clock::now();
    SparseProducts sp; // outlives the fit: the sweeps use its workspace
    int st = sp.prepare(ctx, x_indptr, x_indices, x_values, n, c_indptr, c_indices, c_values, M, d, sigma, (2 * iters + 1) * t);
    if (st) return st;
    knm_precond *p = nullptr;
    st = precond_build_csr_impl(ctx, c_indptr, c_indices, c_values, M, d, sigma, lambda, jitter, true, true, &p, nullptr);
    if (st) return st;
    KernelOps ops;
    ops.n = n;
    ops.M = M;
    ops.v = [&sp](const float *V, int tt, float *W) { return sp.v(V, tt, W); };
    ops.t_w = [&sp](const float *W, const float *wgt, int tt, float *U) { return sp.t_w(W, wgt, tt, U); };
    return fit_core(ctx, ops, p, Y, t, lambda, iters, alpha, resid_norms_or_null, t_start);
}

int knm_v_csr(knm_ctx *ctx, const int64_t *x_indptr, const int64_t *x_indices, const float *x_values, int64_t n,
              const int64_t *c_indptr, const int64_t *c_indices, const float *c_values, int64_t M, int64_t d,
              float sigma, const float *V, int t, float *W)
{
    if (!ctx) return KNM_INVALID_ARG;
    if (!x_indptr || !c_indptr || !V || !W || n <= 0 || M <= 0 || d <= 0 || t <= 0 || !(sigma > 0.0f))
        return fail(ctx, KNM_INVALID_ARG, "bad shape or pointer");
    if (d >= 0x7fffffffLL || M >= 0x7fffffffLL || t > knm_max_t())
        return fail(ctx, KNM_UNSUPPORTED, "d, M or t above the supported maximum");
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipSetDevice");
    SparseProducts sp;
    int st = sp.prepare(ctx, x_indptr, x_indices, x_values, n, c_indptr, c_indices, c_values, M, d, sigma, t);
    if (!st) st = sp.v(V, t, W);
    if (st) return st;
    hipError_t e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "knm_v_csr", e);
    return KNM_OK;
}

int knm_get_fit_timing(const knm_ctx *ctx, double *seconds)
{
    if (!ctx || !seconds) return KNM_INVALID_ARG;
    for (int i = 0; i < 4; ++i) seconds[i] = ctx->fit_seconds[i];
    return KNM_OK;
}

int falkon_predict(knm_ctx *ctx, const float *Xtest, int64_t ntest, int d, int64_t ldx, const float *C, int64_t M,
                   int64_t ldc, float sigma, const float *alpha, int t, float *out)
{
    return knm_v(ctx, Xtest, ntest, d, ldx, C, M, ldc, sigma, alpha, t, out);
}

// Newton iteration of the logistic fit (Alg. 2) on whatever storage the points have: `ops` are the
// two sweeps of k(X, C), `centres_v` gives k(C, C) a (M floats); p holds T (its second factor is
// rebuilt at every step) and is freed on return.
static int logfalkon_core(knm_ctx *ctx, const KernelOps &ops, const std::function<int(const float *, float *)> &centres_v,
                          knm_precond *p, const float *y, const float *yC, const double *lambdas, const int *iters,
                          int n_steps, double jitter, float *alpha, double *loss_or_null)
{
    const int64_t n = ops.n, M = ops.M;
    int st = KNM_OK;
    struct Guard {
        knm_precond *p;
        ~Guard() { precond_free(p); }
    } guard{p};

    const int blocks = red_blocks(M), loss_blocks = kMaxRedBlocks;
    const dim3 vgrid((unsigned)blocks), vblock(256);
    int max_iters = 0;
    for (int k = 0; k < n_steps; ++k) max_iters = iters[k] > max_iters ? iters[k] : max_iters;
    LinopWork wk;
    DevBuf a64, a32, z, zc, g, dw, dm, lossv, beta, r, pv, q, scal, badbuf;
    st = wk.alloc(ctx, M, 1);
    if (!st) st = a64.alloc(ctx, sizeof(double) * M);
    if (!st) st = a32.alloc(ctx, sizeof(float) * M);
    if (!st) st = z.alloc(ctx, sizeof(float) * n);
    if (!st) st = zc.alloc(ctx, sizeof(float) * M);
    if (!st) st = g.alloc(ctx, sizeof(float) * n);
    if (!st) st = dw.alloc(ctx, sizeof(float) * n);
    if (!st) st = dm.alloc(ctx, sizeof(double) * M);
    if (!st && loss_or_null) st = lossv.alloc(ctx, sizeof(double) * n);
    if (!st) st = beta.alloc(ctx, sizeof(double) * M);
    if (!st) st = r.alloc(ctx, sizeof(double) * M);
    if (!st) st = pv.alloc(ctx, sizeof(double) * M);
    if (!st) st = q.alloc(ctx, sizeof(double) * M);
    // mean losses, r . r of every iteration of a step, partials of p . q, of r . r and of the loss
    if (!st) st = scal.alloc(ctx, sizeof(double) * ((size_t)n_steps + 1 + max_iters + 1 + 2 * blocks + loss_blocks));
    if (!st) st = badbuf.alloc(ctx, sizeof(unsigned long long));
    if (st) return st;
    double *da = a64.as<double>(), *db = beta.as<double>(), *dr = r.as<double>(), *dp = pv.as<double>(),
           *dq = q.as<double>();
    double *losses = scal.as<double>(), *rho = losses + n_steps + 1, *part_pq = rho + max_iters + 1, *part_rr = part_pq + blocks,
           *part_loss = part_rr + blocks;
    hipError_t e = hipMemsetAsync(da, 0, sizeof(double) * M, ctx->stream);
    if (e == hipSuccess) e = hipMemsetAsync(a32.p, 0, sizeof(float) * M, ctx->stream);
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipMemsetAsync", e);
    // predictions at the rows for the current alpha and the loss terms, the mean loss to `mean_loss` (device, or null)
    auto evaluate = [&](bool derivatives, double *mean_loss) -> int {
        int s2 = ops.v(a32.as<float>(), 1, z.as<float>());
        if (s2) return s2;
        hipLaunchKernelGGL(logistic_terms_kernel, grid1(n), dim3(256), 0, ctx->stream, z.as<float>(), y, n,
                           derivatives ? g.as<float>() : nullptr, derivatives ? dw.as<float>() : nullptr,
                           (double *)nullptr, mean_loss ? lossv.as<double>() : nullptr);
        if (mean_loss) {
            hipLaunchKernelGGL(dot_partial_kernel, dim3((unsigned)loss_blocks), dim3(256), 0, ctx->stream, lossv.as<double>(),
                               (const double *)nullptr, n, part_loss);
            hipLaunchKernelGGL(dot_finish_kernel, dim3(1), dim3(64), 0, ctx->stream, part_loss, loss_blocks, 1.0 / (double)n, mean_loss);
        }
        return hipGetLastError() == hipSuccess ? KNM_OK : fail(ctx, KNM_HIP_ERROR, "loss terms launch");
    };

    CrossTermScope cross(ctx);
    st = cross.begin();
    if (st) return st;
    for (int k = 0; k < n_steps; ++k) {
        const double mu = lambdas[k];
        st = evaluate(true, loss_or_null ? losses + k : nullptr);
        if (st) return st;
        if (k == 0) {
            bool repeat = false;
            st = cross.check(&repeat);
            if (!st && repeat) st = evaluate(true, loss_or_null ? losses : nullptr);
            if (st) return st;
        }
        // weights at the centres -> second factor of the preconditioner for this step
        st = centres_v(a32.as<float>(), zc.as<float>());
        if (st) return st;
        hipLaunchKernelGGL(logistic_terms_kernel, grid1(M), dim3(256), 0, ctx->stream, zc.as<float>(), yC, M,
                           (float *)nullptr, (float *)nullptr, dm.as<double>(), (double *)nullptr);
        st = build_second_factor(ctx, p, mu, dm.as<double>(), badbuf.as<unsigned long long>());
        if (st) return st;
        // right-hand side  -P^T (K^T g + mu n (K_MM + eps I) alpha)
        st = ops.t_w(g.as<float>(), nullptr, 1, wk.u32.as<float>());
        if (st) return st;
        hipLaunchKernelGGL(newton_rhs_kernel, grid1(M), dim3(256), 0, ctx->stream, wk.u32.as<float>(), zc.as<float>(), da,
                           mu * (double)n, jitter, M, wk.c.as<double>());
        st = tri_solve(ctx, p, p->T, p->Tdinv, true, wk.c.as<double>(), wk.w.as<double>(), 1);
        if (!st) st = tri_solve(ctx, p, p->A, p->Adinv, true, wk.w.as<double>(), dr, 1);
        // (the host looks at the factorisation here, with the work up to the right-hand side already queued)
        int64_t pivot = 0;
        if (!st) st = read_bad_pivots(ctx, badbuf.as<unsigned long long>(), 1, &pivot);
        if (!st && pivot != 0) st = fail(ctx, KNM_NOT_PD, kSecondNotPd);
        if (st) return st;
        e = hipMemsetAsync(db, 0, sizeof(double) * M, ctx->stream);
        if (e == hipSuccess) e = hipMemcpyAsync(dp, dr, sizeof(double) * M, hipMemcpyDeviceToDevice, ctx->stream);
        if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "CG initialisation", e);
        hipLaunchKernelGGL(dot_partial_kernel, vgrid, vblock, 0, ctx->stream, dr, dr, M, part_rr);
        hipLaunchKernelGGL(dot_finish_kernel, dim3(1), dim3(64), 0, ctx->stream, part_rr, blocks, 1.0, rho);
        for (int it = 0; it < iters[k]; ++it) {
            st = linop_cols(ctx, p, wk, ops, mu, dp, 1, dq, dw.as<float>());
            if (st) return st;
            launch_cg_update(ctx->stream, M, 1, rho + it, rho + it + 1, dp, dq, db, dr, part_pq, part_rr);
        }
        // alpha += T^-1 A^-1 beta
        st = tri_solve(ctx, p, p->A, p->Adinv, false, db, wk.v.as<double>(), 1);
        if (!st) st = tri_solve(ctx, p, p->T, p->Tdinv, false, wk.v.as<double>(), wk.w.as<double>(), 1);
        if (st) return st;
        hipLaunchKernelGGL(add_round_kernel, grid1(M), dim3(256), 0, ctx->stream, M, wk.w.as<double>(), da, a32.as<float>());
    }
    if (loss_or_null) {
        st = evaluate(false, losses + n_steps);
        if (st) return st;
        e = hipMemcpyAsync(loss_or_null, losses, sizeof(double) * ((size_t)n_steps + 1), hipMemcpyDeviceToHost, ctx->stream);
    }
    if (e == hipSuccess) e = hipMemcpyAsync(alpha, a32.p, sizeof(float) * M, hipMemcpyDeviceToDevice, ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream); // the caller's arrays are written, the temporaries done with
    if (e == hipSuccess) e = hipGetLastError();
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "logfalkon_fit", e);
    return KNM_OK;
}


int logfalkon_fit(knm_ctx *ctx, const float *X, int64_t n, int d, int64_t ldx, const float *y, const float *C, int64_t M,
                  int64_t ldc, const float *yC, float sigma, const double *lambdas, const int *iters, int n_steps,
                  double jitter, float *alpha, double *loss_or_null)
{
    if (!ctx) return KNM_INVALID_ARG;
    if (!X || !y || !C || !yC || !alpha || !lambdas || !iters || n <= 0 || M <= 0 || d <= 0 || n_steps <= 0 ||
        ldx < d || ldc < d || !(sigma > 0.0f) || !(jitter >= 0.0))
        return fail(ctx, KNM_INVALID_ARG, "bad fit argument");
    for (int k = 0; k < n_steps; ++k)
        if (!(lambdas[k] >= 0.0) || iters[k] <= 0) return fail(ctx, KNM_INVALID_ARG, "bad Newton schedule");
    if (d > knm_max_d()) return fail(ctx, KNM_UNSUPPORTED, "d above compiled maximum");
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipSetDevice");
    int st = KNM_OK;
    // T depends on the centres only: built once; A is rebuilt per Newton step
    knm_precond *p = nullptr;
    st = precond_build_impl(ctx, C, M, d, ldc, sigma, lambdas[0], jitter, false, true, &p, nullptr);
    if (st) return st;
    SweepShare share(ctx, X, n, ldx, C, M, ldc, d, sigma, 1, true);
    for (int k = 0; k < n_steps; ++k) share.uses += 2 * iters[k] + 2;
    const ShareScope scope(share);
    const KernelOps ops = dense_ops(ctx, X, n, d, ldx, C, M, ldc, sigma);
    auto centres_v = [=](const float *a, float *zc) { return do_knm_v(ctx, C, M, d, ldc, C, M, ldc, sigma, a, 1, zc); };
    return logfalkon_core(ctx, ops, centres_v, p, y, yC, lambdas, iters, n_steps, jitter, alpha, loss_or_null);
}

int logfalkon_fit_csr(knm_ctx *ctx, const int64_t *x_indptr, const int64_t *x_indices, const float *x_values, int64_t n,
                      const float *y, const int64_t *c_indptr, const int64_t *c_indices, const float *c_values, int64_t M,
                      int64_t d, const float *yC, float sigma, const double *lambdas, const int *iters, int n_steps,
                      double jitter, float *alpha, double *loss_or_null)
{
    if (!ctx) return KNM_INVALID_ARG;
    if (!x_indptr || !c_indptr || !y || !yC || !alpha || !lambdas || !iters || n <= 0 || M <= 0 || d <= 0 ||
        n_steps <= 0 || !(sigma > 0.0f) || !(jitter >= 0.0))
        return fail(ctx, KNM_INVALID_ARG, "bad fit argument");
    for (int k = 0; k < n_steps; ++k)
        if (!(lambdas[k] >= 0.0) || iters[k] <= 0) return fail(ctx, KNM_INVALID_ARG, "bad Newton schedule");
    if (d >= 0x7fffffffLL || M >= 0x7fffffffLL) return fail(ctx, KNM_UNSUPPORTED, "d or M above the supported maximum");
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipSetDevice");
    // the sweeps of k(X, C) and of k(C, C); both outlive the fit, which uses their workspaces
    SparseProducts sp, spc;
    int st = sp.prepare(ctx, x_indptr, x_indices, x_values, n, c_indptr, c_indices, c_values, M, d, sigma, 2);
    if (!st) st = spc.prepare(ctx, c_indptr, c_indices, c_values, M, c_indptr, c_indices, c_values, M, d, sigma, n_steps);
    if (st) return st;
    knm_precond *p = nullptr;
    st = precond_build_csr_impl(ctx, c_indptr, c_indices, c_values, M, d, sigma, lambdas[0], jitter, false, true, &p, nullptr);
    if (st) return st;
    KernelOps ops;
    ops.n = n;
    ops.M = M;
    ops.v = [&sp](const float *V, int tt, float *W) { return sp.v(V, tt, W); };
    ops.t_w = [&sp](const float *W, const float *wgt, int tt, float *U) { return sp.t_w(W, wgt, tt, U); };
    auto centres_v = [&spc](const float *a, float *zc) { return spc.v(a, 1, zc); };
    return logfalkon_core(ctx, ops, centres_v, p, y, yC, lambdas, iters, n_steps, jitter, alpha, loss_or_null);
}

} // extern "C"
