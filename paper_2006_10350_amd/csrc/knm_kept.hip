// Sums over kept kernel values: out[i, c] = sum_j K[i, j] vec[j, c] (see knm_internal.h for the layout of K).
//
// A fit's, along either side of the matrix, on the fp64 matrix cores: a value is fp32, its products and all sums are fp64.  Bound by the bandwidth of the values, which are read once for up to 16 columns: 60000 x 10000 values with 10 columns in 0.45 ms,
// 5.4 TB/s (0.47 at three workgroups per CU with a second copy of the units in registers).  An instruction of 16 x 16 x 4 takes 64 values
// in 64 cycles: 9.8 TB/s over the chip, half of that with 17 to 32 columns.  The sweep that forms the values anew takes 1.85 ms at d = 784.
#include <type_traits>

#include "knm_internal.h"
#include "knm_operands.h"

namespace knm {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int workgroups_per_cu(int g) { return g == 1 ? 4 : 2; } // by registers

struct SumArgs {
    KeptArgs k;
    int64_t n_s32;      // stream blocks of 32
    int64_t in_blocks;  // blocks of 32 points summed over
    int64_t chunk;      // of them per chunk
    int64_t n_in, n_out;
};

// Entries of 16 rows of the vectors on their way from memory: rows r0 + STEP e + at, columns 16 g + l % 16 (a column that
// does not exist takes the last one, and its sums are not stored).  Rows past the end are zero.
template <int G, int STEP, bool WGT> struct Entries {
    float v[4][G], w[WGT ? 4 : 1];
    int left; // rows there are
    __device__ __forceinline__ void load(const SumArgs &a, int64_t r0, int at, const int (&col)[G])
    {
        left = a.n_in - r0 >= 16 ? 16 : (int)(a.n_in - r0);
        const int64_t r0c = left > 0 ? r0 : 0;
        const float *const vec = a.k.vec + r0c * a.k.t;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int r = STEP * e + at < left ? STEP * e + at : 0;
#pragma unroll
            for (int g = 0; g < G; ++g) v[e][g] = vec[r * a.k.t + col[g]];
            if constexpr (WGT) w[e] = a.k.wgt[r0c + r];
        }
    }
    __device__ __forceinline__ double value(int e, int g, int at) const
    {
        const float p = WGT ? v[e][g] * w[e] : v[e][g];
        return STEP * e + at < left ? (double)p : 0.0;
    }
};
__device__ __forceinline__ void store_sum(const SumArgs &a, int64_t i, int c, double v)
{
    if (i >= a.n_out || c >= a.k.t) return;
    a.k.part[((int64_t)blockIdx.y * a.n_out + i) * a.k.t + c] = v;
}

// (the wavefront's number in the grid's first dimension, as a scalar)
__device__ __forceinline__ int64_t wavefront()
{
    return (int64_t)blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}

// Sum over the stream points.  A wavefront has 64 fixed points, four 16-row tiles; lane l holds fixed point l % 16 of
// a tile and, in one unit, stream rows 16 j + 4 (l / 16) + e of the block: the A operand of product e.  Half a block is loaded
// while the other half is multiplied.
template <int G, bool WGT>
__global__ __launch_bounds__(kThreads, workgroups_per_cu(G)) void kept_over_stream_kernel(SumArgs a)
{
    const int lane = threadIdx.x & 63, l15 = lane & 15, q = lane >> 4;
    const int64_t fixed0 = wavefront() * 64;
    const int64_t b0 = (int64_t)blockIdx.y * a.chunk;
    const int64_t b1 = b0 + a.chunk < a.in_blocks ? b0 + a.chunk : a.in_blocks;
    const float *const base = a.k.values + (fixed0 >> 5) * a.n_s32 * kKeptBlock;
    const int at = (kept_unit(l15, 0) + 4 * q) * 4;
    int col[G];
#pragma unroll
    for (int g = 0; g < G; ++g) col[g] = 16 * g + l15 < a.k.t ? 16 * g + l15 : a.k.t - 1;
    f64x4 acc[4][G];
#pragma unroll
    for (int f = 0; f < 4; ++f)
#pragma unroll
        for (int g = 0; g < G; ++g) acc[f][g] = f64x4{0.0, 0.0, 0.0, 0.0};
    f32x4 kv[2][4];
    Entries<G, 1, WGT> v[2];
    // half j of block b: units (rq, h) = 4 j + q of fixed points l15 (+ 16) of two fixed blocks
    auto load = [&](int64_t b, int j) {
#pragma unroll
        for (int f = 0; f < 4; ++f)
            kv[j][f] = *reinterpret_cast<const f32x4 *>(base + ((f >> 1) * a.n_s32 + b) * kKeptBlock + (f & 1) * 512 + j * 64 + at);
        v[j].load(a, b * 32 + 16 * j, 4 * q, col);
    };
    if (b0 < b1) {
        load(b0, 0);
        load(b0, 1);
    }
    for (int64_t b = b0; b < b1; ++b) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                double bv[G];
#pragma unroll
                for (int g = 0; g < G; ++g) bv[g] = v[j].value(e, g, 4 * q);
#pragma unroll
                for (int f = 0; f < 4; ++f)
#pragma unroll
                    for (int g = 0; g < G; ++g)
                        acc[f][g] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)kv[j][f][e], bv[g], acc[f][g], 0, 0, 0);
            }
            if (b + 1 < b1) load(b + 1, j);
        }
    }
#pragma unroll
    for (int f = 0; f < 4; ++f)
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int r = 0; r < 4; ++r) store_sum(a, fixed0 + 16 * f + 4 * r + q, 16 * g + l15, acc[f][g][r]);
}

// Sum over the fixed points.  A wavefront has 64 stream points; lane l holds, in one unit, the four rows 4 (l % 16) + e of them for
// fixed point l / 16 of four: product e gives the rows 4 i + e.
template <int G, bool WGT>
__global__ __launch_bounds__(kThreads, workgroups_per_cu(G)) void kept_over_fixed_kernel(SumArgs a)
{
    const int lane = threadIdx.x & 63, l15 = lane & 15, q = lane >> 4;
    const int64_t s32 = wavefront() * 2;
    if (s32 >= a.n_s32) return; // (n_s32 is a multiple of 4)
    const int64_t b0 = (int64_t)blockIdx.y * a.chunk;
    const int64_t b1 = b0 + a.chunk < a.in_blocks ? b0 + a.chunk : a.in_blocks;
    const float *const base = a.k.values + s32 * kKeptBlock;
    const int at = (l15 >> 3) * kKeptBlock + ((l15 & 7) * 4 + q) * 4;
    int col[G];
#pragma unroll
    for (int g = 0; g < G; ++g) col[g] = 16 * g + l15 < a.k.t ? 16 * g + l15 : a.k.t - 1;
    f64x4 acc[4][G];
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int g = 0; g < G; ++g) acc[e][g] = f64x4{0.0, 0.0, 0.0, 0.0};
    f32x4 kv[2][4];
    Entries<G, 4, WGT> v[2];
    // fixed points 16 j + 4 i + q of block b, i < 4
    auto load = [&](int64_t b, int j) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            kv[j][i] = *reinterpret_cast<const f32x4 *>(base + b * a.n_s32 * kKeptBlock + (4 * j + i) * 128 + at);
        v[j].load(a, b * 32 + 16 * j, q, col);
    };
    if (b0 < b1) {
        load(b0, 0);
        load(b0, 1);
    }
    for (int64_t b = b0; b < b1; ++b) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                double bv[G];
#pragma unroll
                for (int g = 0; g < G; ++g) bv[g] = v[j].value(i, g, q);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int g = 0; g < G; ++g)
                        acc[e][g] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)kv[j][i][e], bv[g], acc[e][g], 0, 0, 0);
            }
            if (b + 1 < b1) load(b + 1, j);
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int r = 0; r < 4; ++r) store_sum(a, s32 * 32 + 4 * (4 * r + q) + e, 16 * g + l15, acc[e][g][r]);
}

// Sums over kept rows (KeptRowsArgs) with fp32 matrix instructions, of which one of 16 x 16 x 4 adds its four products to an entry one
// after the other, each with one rounding: what the vector ALU of the engine does for four consecutive rows.  A wavefront has 64
// centres, one half h of the rows and up to 16 columns; lane l holds, in one unit, centres 4 (l % 16) ... + 3 for row l / 16 of four,
// and product e is that of centres 4 i + e.  A workgroup is two groups of centres and both halves, over the part of one
// chunk that lies in the slab: the order of a chunk's sums is fixed, so the chunks and the centres are all there is to share
// out, and a wavefront has a whole tile (16 KB) on its way.  Bound by the bandwidth of the values: 16384 x 50000 of them, 10 columns, in
// 0.53 ms, 6.2 TB/s (0.63 with loads that leave the values in the caches; on the vector ALU, one lane per centre, with the vector entries from
// scalar loads 1.3 to 1.6 ms: they came from the L2).
__global__ __launch_bounds__(kThreads, 2) void kept_rows_kernel(KeptRowsArgs a, int64_t n_s32, int64_t chunk0)
{
    __shared__ double other[2][16][64];
    const int lane = threadIdx.x & 63, l15 = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int h = wave & 1, pair = wave >> 1;
    const int64_t s0 = ((int64_t)blockIdx.x * 2 + pair) * 64; // (n_s32 is even: both blocks of 32 exist or neither)
    const int64_t chunk = chunk0 + blockIdx.y;
    const int64_t chunk_begin = chunk * a.chunk_len;
    const int64_t begin = chunk_begin > a.row0 ? chunk_begin : a.row0;
    const int64_t slab_end = a.row0 + a.rows;
    const int64_t chunk_end = chunk_begin + a.chunk_len < a.n ? chunk_begin + a.chunk_len : a.n;
    const int64_t end = chunk_end < slab_end ? chunk_end : slab_end;
    const int col = l15 < a.t ? l15 : a.t - 1; // (a column that does not exist repeats the last one and is not stored)
    // entry (e, r) of this lane: centre s0 + 4 (4 r + q) + e, column l15
    auto stored = [&](int e, int r) { return l15 < a.t && s0 + 4 * (4 * q + r) + e < a.nS; };
    auto state_at = [&](int e, int r) { return ((int64_t)h * a.nS + s0 + 4 * (4 * q + r) + e) * a.t + l15; };
    f32x4 sum[4];
    double wide[4][4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        sum[e] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int r = 0; r < 4; ++r) wide[e][r] = begin > chunk_begin && stored(e, r) ? a.state_in[state_at(e, r)] : 0.0;
    }
    if ((s0 >> 5) < n_s32 && begin < end) {
        const float *const base = a.values + (s0 >> 5) * kKeptBlock + h * 128;
        const int at = (l15 >> 3) * kKeptBlock + ((l15 & 7) * 4 + q) * 4;
        constexpr int kQuads = kKeptTile / 8; // of a half's rows in a tile
        f32x4 kv[kQuads];
        float w[kQuads];
        // rows `row` + 8 i + 4 h + q, i = 4 b ... 4 b + 3
        auto load = [&](int b, int64_t row) {
            const float *const p = base + (((row - a.row0) >> 5) + b) * n_s32 * kKeptBlock;
            const int left = (int)(end - row < kKeptTile ? end - row : kKeptTile);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = 32 * b + 8 * i + 4 * h + q;
                // (a block of 32 rows that begins past the end does not exist)
                kv[4 * b + i] = __builtin_nontemporal_load(
                    reinterpret_cast<const f32x4 *>((32 * b < left ? p : base + ((row - a.row0) >> 5) * n_s32 * kKeptBlock) + i * 256 + at));
                w[4 * b + i] = a.vec[(row - a.row0 + (r < left ? r : 0)) * a.t + col];
            }
        };
#pragma unroll
        for (int b = 0; b < 4; ++b) load(b, begin);
        for (int64_t row = begin; row < end; row += kKeptTile) {
            const int left = (int)(end - row < kKeptTile ? end - row : kKeptTile);
#pragma unroll
            for (int b = 0; b < 4; ++b) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float wi = 32 * b + 8 * i + 4 * h + q < left ? w[4 * b + i] : 0.0f; // rows past the end add nothing
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[4 * b + i][e], wi, sum[e], 0, 0, 0);
                }
                if (row + kKeptTile < end) load(b, row + kKeptTile);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
#pragma unroll
                for (int r = 0; r < 4; ++r) wide[e][r] += (double)sum[e][r];
                sum[e] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            }
        }
    }
    if (end < chunk_end) { // the chunk goes on in the next slab (the same for all workgroups of a chunk)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (stored(e, r)) a.state_out[state_at(e, r)] = wide[e][r];
        return;
    }
    if (h == 1)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int r = 0; r < 4; ++r) other[pair][4 * e + r][lane] = wide[e][r];
    __syncthreads();
    if (h == 0)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (stored(e, r))
                    a.part[(chunk * a.nS + s0 + 4 * (4 * q + r) + e) * a.t + l15] = (float)(wide[e][r] + other[pair][4 * e + r][lane]);
}

SumArgs sum_args(const KeptArgs &k)
{
    SumArgs a;
    a.k = k;
    a.n_s32 = kept_stream_blocks(k.nS);
    a.in_blocks = k.over_stream ? (k.nS + 31) / 32 : (k.nF + 31) / 32;
    a.n_in = k.over_stream ? k.nS : k.nF;
    a.n_out = k.over_stream ? k.nF : k.nS;
    a.chunk = (a.in_blocks + k.chunks - 1) / k.chunks;
    return a;
}
int64_t workgroups(const SumArgs &a)
{
    const int64_t per = kWaves * 64;
    return (a.n_out + per - 1) / per;
}

} // namespace

int kept_max_t() { return 32; }

// The fewest chunks that fill the places of the chip to 95 %, or as well as up to four rounds of them can: all workgroups are equal, and
// part of a round costs a whole one (50048 x 16384 values: 588 workgroups on 768 places 0.82 ms, 2940 0.68 ms).
int kept_chunks(int64_t nF, int64_t nS, bool over_stream, int t)
{
    KeptArgs k{};
    k.nF = nF;
    k.nS = nS;
    k.over_stream = over_stream;
    k.t = t;
    k.chunks = 1;
    const SumArgs a = sum_args(k);
    const int64_t wgs = workgroups(a), places = 256 * workgroups_per_cu(t <= 16 ? 1 : 2);
    int64_t best = 1;
    double best_fill = 0.0;
    for (int64_t c = 1; c <= a.in_blocks && (c == 1 || c * wgs <= 4 * places) && best_fill < 0.95; ++c) {
        const int64_t rounds = (c * wgs + places - 1) / places;
        const double fill = (double)(c * wgs) / (double)(rounds * places);
        if (fill > best_fill + 0.02) {
            best = c;
            best_fill = fill;
        }
    }
    const int64_t len = (a.in_blocks + best - 1) / best;
    return (int)((a.in_blocks + len - 1) / len);
}

hipError_t launch_kept_sum(const KeptArgs &k, hipStream_t stream)
{
    if (k.nF <= 0 || k.nS <= 0 || k.t <= 0 || k.t > kept_max_t() || k.chunks <= 0 || k.values == nullptr || k.part == nullptr)
        return hipErrorInvalidValue;
    const SumArgs a = sum_args(k);
    const int64_t wgs = workgroups(a);
    if (wgs > 0x7fffff || k.chunks > 65535) return hipErrorInvalidValue;
    const dim3 grid((unsigned)wgs, (unsigned)k.chunks);
    auto launch = [&](auto weighted) {
        constexpr bool W = decltype(weighted)::value;
        auto *kernel = k.over_stream ? (k.t <= 16 ? kept_over_stream_kernel<1, W> : kept_over_stream_kernel<2, W>)
                                     : (k.t <= 16 ? kept_over_fixed_kernel<1, W> : kept_over_fixed_kernel<2, W>);
        hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, stream, a);
    };
    if (k.wgt != nullptr) launch(std::true_type{});
    else launch(std::false_type{});
    return hipGetLastError();
}

hipError_t launch_kept_rows(const KeptRowsArgs &a, hipStream_t stream)
{
    if (a.values == nullptr || a.state_in == nullptr || a.state_out == nullptr || a.part == nullptr || a.t <= 0 || a.t > kept_rows_max_t() || a.rows <= 0 || a.nS <= 0 ||
        a.row0 % 256 != 0 || a.row0 + a.rows > a.n || a.chunk_len <= 0 || a.chunk_len % kKeptTile != 0)
        return hipErrorInvalidValue;
    const int64_t chunk0 = a.row0 / a.chunk_len, chunks = (a.row0 + a.rows + a.chunk_len - 1) / a.chunk_len - chunk0;
    const int64_t wgs = (a.nS + 127) / 128;
    if (wgs > 0x7fffff || chunks > 65535) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kept_rows_kernel, dim3((unsigned)wgs, (unsigned)chunks), dim3(kThreads), 0, stream, a, kept_stream_blocks(a.nS), chunk0);
    return hipGetLastError();
}

} // namespace knm
