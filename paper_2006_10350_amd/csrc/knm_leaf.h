// The leaf of the blocked Cholesky factorisations, a workgroup's work: on its own (knm_solver.hip) or beside the update of the rows it
// belongs to (knm_dsyrk.hip).
#pragma once

#include "knm_internal.h"

namespace knm {

// ---- leaf of the blocked factorisation --------------------------------------------------------
// One workgroup factorises a diagonal block of order nb <= 128 in LDS and inverts the factor there;
// everything above the leaf is products with these small inverses on the matrix cores.
//
// A leaf is a serial chain, one workgroup with the rest of the chip waiting or (look-ahead) busy with
// the trailing update, so what counts is its latency.  The block is cut into 16 x 16 tiles, held as accumulators of
// v_mfma_f64_16x16x4: register r of lane l is entry (4 r + l / 16, l % 16).  Wavefront 0 runs the chain of the diagonal
// tiles: 4 pivots at a time, the 4 x 4 block is read from the lanes as scalars, factorised and inverted by every lane, one
// product with that inverse finishes the 4 rows (register r of the tile, which is at once the operand layout of both sides of
// the rank-4 update that follows, so nothing moves between lanes), and the same products turn the identity into the inverse of
// the tile.  The row of tiles is then multiplied by the inverse, wavefront 0 keeping the tile it needs for the
// next diagonal tile in registers and going on with that one, while the others update the trailing tiles and prepare the next
// column of the inverse, W(:, p) = -(W R(:, p)) W(p, p), up to the factor that the diagonal tile in hand will give: when
// the last diagonal tile is done, the whole inverse is one product away.  Two barriers per tile row.
// 26 us per 128 x 128 block; inverses merged pair by pair at the end 31 us; one column per lane, multipliers read from
// lanes pivot by pivot, 60 us; eliminating row by row from LDS with two barriers per pivot 347 us.
// The kernel keeps to 74 KB of LDS so that it can share a CU with a workgroup of the rank-k
// kernel: during the factorisation's look-ahead it runs beside the trailing update.
constexpr int kLeaf = 128; // LeafArgs::nb at most
constexpr int kLeafThreads = 512;
constexpr int kLeafWaves = kLeafThreads / 64;
constexpr int kLeafTiles = kLeaf / 16;
constexpr int kLeafPairs = kLeafTiles * (kLeafTiles + 1) / 2; // tiles of the upper triangle
constexpr int kLeafDoubles = (kLeafPairs + 1) * 256;

typedef double leaf_d4 __attribute__((ext_vector_type(4)));

// 16 x 16 tile (bi, bj), bi <= bj, of the upper triangle; entry (i, j) of a tile at i 16 + (j ^ i): rows and columns
// are both read without bank conflicts
__host__ __device__ constexpr int leaf_tile(int bi, int bj) { return (bj * (bj + 1) / 2 + bi) * 256; }
__device__ __forceinline__ int leaf_at(int i, int j) { return i * 16 + (j ^ i); }
__host__ __device__ constexpr int leaf_tile_col(int tile)
{
    int bj = 0;
    while ((bj + 1) * (bj + 2) / 2 <= tile) ++bj;
    return bj;
}

__device__ __forceinline__ double lane_value(double x, int lane)
{
    const uint64_t v = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), lane);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// 1 / sqrt(d) for a normal positive d: the hardware's estimate (about 26 bits) and one third-order Newton step
__device__ __forceinline__ double inverse_sqrt(double d)
{
    const double y = __builtin_amdgcn_rsq(d);
    const double e = fma(-(d * y), y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// A^T B or (transposed B) A^T B^T of two 16 x 16 tiles of LDS: operands, and c (accumulator layout) += the product
struct LeafOperands {
    double a[4], b[4];
    template <bool TRANS_B> __device__ __forceinline__ void load(const double *A, const double *B, int lane)
    {
        const int l15 = lane & 15, q = lane >> 4;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int k = 4 * s + q;
            a[s] = A[leaf_at(k, l15)];
            b[s] = TRANS_B ? B[leaf_at(l15, k)] : B[leaf_at(k, l15)];
        }
    }
    __device__ __forceinline__ void multiply(leaf_d4 &c) const
    {
#pragma unroll
        for (int s = 0; s < 4; ++s) c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], c, 0, 0, 0);
    }
};

// Factorises the diagonal tile `acc` (entries on and above its diagonal; what is below only ever reaches entries below):
// rows[r] <- rows 4 r .. 4 r + 3 of R, inv[r] <- the same rows of L^-1 = R^-T, w <- 1 / diagonal of R: NaN from the first
// pivot on that is not a positive finite number.
__device__ __forceinline__ void leaf_diagonal(leaf_d4 acc, leaf_d4 &rows, leaf_d4 &inv_rows, double (&w)[16], int lane)
{
    const int l15 = lane & 15, q = lane >> 4;
    const leaf_d4 zero = {0.0, 0.0, 0.0, 0.0};
    leaf_d4 inv;
#pragma unroll
    for (int r = 0; r < 4; ++r) inv[r] = (4 * r + q == l15) ? 1.0 : 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        double g[4][4], d[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = i; j < 4; ++j) g[i][j] = lane_value(acc[r], 16 * i + 4 * r + j);
#pragma unroll
        for (int i = 0; i < 4; ++i) { // row i of the 4 x 4 factor over g, w its diagonal's inverses
            d[i] = g[i][i];
#pragma unroll
            for (int k = 0; k < i; ++k) d[i] = fma(-g[k][i], g[k][i], d[i]);
            w[4 * r + i] = inverse_sqrt(d[i]);
#pragma unroll
            for (int j = i + 1; j < 4; ++j) {
                double v = g[i][j];
#pragma unroll
                for (int k = 0; k < i; ++k) v = fma(-g[k][i], g[k][j], v);
                g[i][j] = v * w[4 * r + i];
            }
        }
        // X = its inverse transpose (lower triangle): column l / 16 in this lane, by forward substitution, then entry
        // X[l % 16][l / 16] for l % 16 < 4 (the other rows of the products below are not used)
        double x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            double v = (i == q) ? 1.0 : 0.0;
#pragma unroll
            for (int k = 0; k < i; ++k) v = fma(-g[k][i], x[k], v);
            x[i] = v * w[4 * r + i];
        }
        const double xv = l15 == 0 ? x[0] : l15 == 1 ? x[1] : l15 == 2 ? x[2] : x[3];
        // rows 0 .. 3 of the products are their register 0; the products of the inverse run behind the chain
        const leaf_d4 rr = __builtin_amdgcn_mfma_f64_16x16x4f64(xv, acc[r], zero, 0, 0, 0);
        rows[r] = rr[0];
        if (r < 3) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-rr[0], rr[0], acc, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        const leaf_d4 ii = __builtin_amdgcn_mfma_f64_16x16x4f64(xv, inv[r], zero, 0, 0, 0);
        inv_rows[r] = ii[0];
        if (r < 3) inv = __builtin_amdgcn_mfma_f64_16x16x4f64(-rr[0], ii[0], inv, 0, 0, 0);
    }
}

// Triangle of the nb x nb block at A (upper storage: entry (i, j), i <= j, at A[i + j lda]; lower storage: at
// A[j + i lda]) <- its upper Cholesky factor R, R^T R = A, in the same storage; W <- R^-1 (nb x nb, always
// column-major with leading dimension ldw; the 16 x 16 tiles below the diagonal are left as they are: the caller has cleared
// them).  *bad <- min(*bad, pivot0 + k + 1) for a pivot
// k that is not a positive finite number (NaNs from there on; the caller discards the result).
// By a workgroup of kLeafThreads threads, in kLeafDoubles entries of LDS.
__device__ __forceinline__ void leaf_block(const LeafArgs &l, double *sh)
{
    double *const A = l.A, *const W = l.W;
    const int64_t lda = l.lda, ldw = l.ldw, pivot0 = l.pivot0;
    const int nb = l.nb, lower = l.lower;
    unsigned long long *const bad = l.bad;
    constexpr int kRows = kLeafPairs * 256; // the diagonal tile of R just finished, in a tile's layout
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int l15 = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = __builtin_amdgcn_readfirstlane(tid >> 8);
    const int nt = (nb + 15) / 16; // tiles per side; the last one is padded with the identity
    const int64_t row_step = lower ? lda : 1, col_step = lower ? 1 : lda; // of an entry of A
    constexpr int kPasses = kLeafPairs / 2; // two tiles at a time, 16 consecutive threads along the contiguous index
    {
        const int u = tid & 15, v = (tid >> 4) & 15;
        const int i = lower ? v : u, j = lower ? u : v;
        const double *src = A + i * row_step + j * col_step;
        double x[kPasses];
#pragma unroll
        for (int k = 0; k < kPasses; ++k) {
            const int bj = half ? leaf_tile_col(2 * k + 1) : leaf_tile_col(2 * k);
            const int bi = 2 * k + half - bj * (bj + 1) / 2;
            const bool diagonal = bi == bj;
            x[k] = (diagonal && i == j) ? 1.0 : 0.0;
            if ((!diagonal || i <= j) && bj * 16 + j < nb) x[k] = src[16 * (bi * row_step + bj * col_step)];
        }
#pragma unroll
        for (int k = 0; k < kPasses; ++k) sh[(2 * k + half) * 256 + leaf_at(i, j)] = x[k];
    }
    __syncthreads();
    auto read_tile = [&](leaf_d4 &c, int at) {
#pragma unroll
        for (int r = 0; r < 4; ++r) c[r] = sh[at + leaf_at(4 * r + q, l15)];
    };
    auto write_tile = [&](int at, const leaf_d4 &c) {
#pragma unroll
        for (int r = 0; r < 4; ++r) sh[at + leaf_at(4 * r + q, l15)] = c[r];
    };
    auto write_out = [&](int bi, int bj, const leaf_d4 &c) { // a tile of R
        const int col = bj * 16 + l15;
        double *dst = A + (bi * 16 + q) * row_step + col * col_step;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (bi * 16 + 4 * r + q <= col && col < nb) dst[4 * r * row_step] = c[r];
    };
    leaf_d4 diag = {0.0, 0.0, 0.0, 0.0}; // wavefront 0: the diagonal tile of the row in hand
    if (wave == 0) read_tile(diag, 0);
    const int ui = wave - 1; // the other wavefronts: row of the inverse whose entry in column p they prepare, for ui < p
    for (int p = 0; p < nt; ++p) {
        leaf_d4 rows, u = {0.0, 0.0, 0.0, 0.0};
        if (wave == 0) {
            leaf_d4 inv;
            double w[16];
            leaf_diagonal(diag, rows, inv, w, lane);
            if (w[15] != w[15]) { // the first failing pivot
                int first = 15;
#pragma unroll
                for (int k = 14; k >= 0; --k) first = w[k] != w[k] ? k : first;
                if (lane == 0) atomicMin(bad, (unsigned long long)(pivot0 + 16 * p + first + 1));
            }
            // the inverse takes the place of the tile
#pragma unroll
            for (int r = 0; r < 4; ++r) sh[leaf_tile(p, p) + leaf_at(l15, 4 * r + q)] = inv[r];
            write_tile(kRows, rows);
        } else if (p > 0) {
            // wavefront 0's tile of R goes out from LDS
            if (wave == kLeafWaves - 1) {
                leaf_d4 c;
                read_tile(c, leaf_tile(p - 1, p));
                write_out(p - 1, p, c);
            }
            // the trailing tiles lose R_p-1,ti^T R_p-1,tj
            const int rest = nt - p, tiles = rest * (rest + 1) / 2;
            for (int t = kLeafWaves - wave; t < tiles; t += kLeafWaves - 1) { // (tile 0 is wavefront 0's)
                int cj = 0;
                while ((cj + 1) * (cj + 2) / 2 <= t) ++cj;
                const int tj = p + cj, ti = p + t - cj * (cj + 1) / 2;
                LeafOperands ops;
                leaf_d4 c = {0.0, 0.0, 0.0, 0.0}, old;
                ops.load<false>(sh + leaf_tile(p - 1, ti), sh + leaf_tile(p - 1, tj), lane);
                read_tile(old, leaf_tile(ti, tj));
                ops.multiply(c);
                write_tile(leaf_tile(ti, tj), old - c);
            }
            // u = (sum_k W(ui, k) R(k, p))^T, which is the operand layout of its next product
            if (ui < p) {
                LeafOperands ops[2];
                ops[0].load<true>(sh + leaf_tile(ui, p), sh + leaf_tile(ui, ui), lane);
                for (int k = ui; k < p; k += 2) {
                    if (k + 1 < p) ops[1].load<true>(sh + leaf_tile(k + 1, p), sh + leaf_tile(ui, k + 1), lane);
                    ops[0].multiply(u);
                    if (k + 1 < p) {
                        if (k + 2 < p) ops[0].load<true>(sh + leaf_tile(k + 2, p), sh + leaf_tile(ui, k + 2), lane);
                        ops[1].multiply(u);
                    }
                }
            }
        }
        __syncthreads();
        // the tiles to the right, R_p,bj = L^-1 A_p,bj, and the column of the inverse
        const int bj = wave == 0 ? p + 1 : wave + 1;
        const bool solve = bj < nt && (wave == 0 || ui >= p);
        leaf_d4 c = {0.0, 0.0, 0.0, 0.0}, next = {0.0, 0.0, 0.0, 0.0}, done = {0.0, 0.0, 0.0, 0.0};
        if (wave == kLeafWaves - 1) read_tile(done, kRows);
        if (solve) {
            LeafOperands ops;
            ops.load<false>(sh + leaf_tile(p, p), sh + leaf_tile(p, bj), lane);
            if (wave == 0) read_tile(next, leaf_tile(p + 1, p + 1));
            ops.multiply(c);
            write_tile(leaf_tile(p, bj), c);
        } else if (wave > 0 && ui < p) {
            LeafOperands ops;
            ops.load<false>(sh + leaf_tile(p, p), sh + leaf_tile(p, p), lane);
#pragma unroll
            for (int s = 0; s < 4; ++s) ops.a[s] = -u[s];
            ops.multiply(c);
            write_tile(leaf_tile(ui, p), c);
        }
        __syncthreads();
        if (wave == kLeafWaves - 1) write_out(p, p, done); // the diagonal tile of R
        if (solve && wave > 0) write_out(p, bj, c);
        if (wave == 0) {
            // the next diagonal tile, from registers
            diag = next;
#pragma unroll
            for (int r = 0; r < 4; ++r) diag = __builtin_amdgcn_mfma_f64_16x16x4f64(-c[r], c[r], diag, 0, 0, 0);
        }
    }
    {
        const int i = tid & 15, j = (tid >> 4) & 15;
#pragma unroll
        for (int k = 0; k < kPasses; ++k) {
            const int bj = half ? leaf_tile_col(2 * k + 1) : leaf_tile_col(2 * k);
            const int bi = 2 * k + half - bj * (bj + 1) / 2;
            const int gi = bi * 16 + i, gj = bj * 16 + j;
            if (gi < nb && gj < nb) W[gi + gj * ldw] = sh[(2 * k + half) * 256 + leaf_at(i, j)];
        }
    }
}

} // namespace knm
