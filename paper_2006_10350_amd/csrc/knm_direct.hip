// Small predictions: W[i, c] = sum_j k(x_i, c_j) V[j, c] in one launch, the kernel values from fp32 differences of the two rows.
//
// A call on a few hundred rows and a thousand centres is all launches: common shift, packed image, sweep and merge took 22 us for 200
// x 1000 values of 8 features, of which the arithmetic is 1.  From differences there are no norms, hence nothing to prepare, no range
// limit and no second evaluation of near pairs.  A thread has one centre at a time and R rows, whose features come from LDS as
// broadcasts; it adds at most kCentresPerThread terms in fp32, a workgroup's threads are added in fp32 over a wavefront and in
// fp64 beyond it, and so are the parts of a row that is split over several workgroups (launch_merge).
#include <limits>
#include <type_traits>

#include "knm_internal.h"
#include "knm_operands.h"

namespace knm {
namespace {

constexpr int kThreads = 256;
constexpr int kCentresPerThread = 16;
constexpr int kChunk = kThreads * kCentresPerThread; // centres of a workgroup at most
constexpr int kMaxD = 128;

struct DirectArgs {
    const float *X, *C, *V;
    int64_t n, ldx, M, ldc;
    int d, t;
    float s2;     // of the engines' sigma
    int chunk;    // centres per workgroup
    float *out;   // n x t
    double *part; // chunks x n x t, or null
    unsigned int *range_count; // as SweepArgs has it, or null
    float inv2s2;              // of the caller's sigma
    float most;                // exponents are no larger, nor a NaN where this is none
};
constexpr int kSample = 16384; // rows that the engines' common shift is the mean of, at most

// A program that asks knm_range_exceeded hears of the points that the split-fp16 engines could not take, though nothing is clamped here.  The
// engines measure from their common shift, the mean of the smaller set (nothing, where that is less than one sigma), which this path does not
// have.  A point more than the range from the shift is at least that far from some point of the smaller set, and every point of the other set is
// more than a third of the range from one of the two.  So a workgroup that sees such a distance, between any of its rows and
// centres, forms the shift and measures its own points and the whole smaller set from there; usual data never gets there.
template <int R> __device__ __forceinline__ void count_out_of_range(const DirectArgs &a, int64_t row0, int64_t j0, int64_t j1)
{
    __shared__ double sums[kThreads];
    __shared__ float mu[kMaxD];
    __shared__ bool shifted;
    const int tid = threadIdx.x;
    const bool rows = a.n <= a.M; // the smaller set
    const float *const P = rows ? a.X : a.C;
    const int64_t count = rows ? a.n : a.M, ld = rows ? a.ldx : a.ldc;
    const int64_t stride = (count + kSample - 1) / kSample;
    const int sample = (int)((count + stride - 1) / stride);
    const int bits = a.d <= 1 ? 0 : 32 - __clz(a.d - 1);
    const int f = tid & ((1 << bits) - 1);
    double s = 0.0;
    if (f < a.d)
        for (int r = tid >> bits; r < sample; r += kThreads >> bits) s += (double)P[r * stride * ld + f];
    sums[tid] = s;
    __syncthreads();
    if (tid < a.d) {
        for (int k = tid + (1 << bits); k < kThreads; k += 1 << bits) s += sums[k];
        const float m = (float)(s / (double)sample);
        mu[tid] = (m == m && fabsf(m) < 3.0e38f) ? m : 0.0f;
    }
    __syncthreads();
    if (tid == 0) {
        double sq = 0.0;
        for (int k = 0; k < a.d; ++k) sq += (double)mu[k] * (double)mu[k];
        shifted = sq * (double)a.inv2s2 > 0.5;
    }
    __syncthreads();
    bool beyond = false;
    auto check = [&](const float *points, int64_t ldp, int64_t begin, int64_t end) {
        for (int64_t i = begin + tid; i < end; i += kThreads) {
            float q = 0.0f;
            for (int k = 0; k < a.d; ++k) {
                const float diff = points[i * ldp + k] - (shifted ? mu[k] : 0.0f);
                q = fmaf(diff, diff, q);
            }
            beyond |= !(a.s2 * q <= kNormMax);
        }
    };
    check(P, ld, 0, count);
    if (rows) check(a.C, a.ldc, j0, j1);
    else check(a.X, a.ldx, row0, row0 + R < a.n ? row0 + R : a.n);
    if (__syncthreads_or(beyond) && tid == 0) atomicAdd(a.range_count, 1u);
}

// R rows, TP columns; VW = 4: the rows of both sets can be read 16 bytes at a time
template <int KIND, int R, int TP, int VW>
__global__ __launch_bounds__(kThreads) void direct_kernel(DirectArgs a)
{
    __shared__ __attribute__((aligned(16))) float xs[kMaxD / 4][R][4];
    __shared__ float red[kThreads / 64][R * TP];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t row0 = (int64_t)blockIdx.x * R;
    const int d4 = (a.d + 3) / 4;
    for (int k = tid; k < d4 * 4 * R; k += kThreads) {
        const int r = k / (d4 * 4), f = k % (d4 * 4);
        const int64_t row = row0 + r < a.n ? row0 + r : a.n - 1; // (a row that does not exist repeats the last one and is not stored)
        const float v = a.X[f < a.d ? row * a.ldx + f : 0];
        xs[f >> 2][r][f & 3] = f < a.d ? v : 0.0f; // (features past the last are zero on both sides)
    }
    __syncthreads();
    const int64_t j0 = (int64_t)blockIdx.y * a.chunk, j1 = j0 + a.chunk < a.M ? j0 + a.chunk : a.M;
    float sum[R][TP];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < TP; ++c) sum[r][c] = 0.0f;
    unsigned farthest = 0; // bits of the largest q: squares order like their bit patterns, and a NaN lies above all of them
    for (int64_t j = j0 + tid; j < j1; j += kThreads) {
        const float *cj = a.C + j * a.ldc;
        float v[TP], q[R];
#pragma unroll
        for (int c = 0; c < TP; ++c) v[c] = a.V[j * a.t + (c < a.t ? c : 0)];
#pragma unroll
        for (int r = 0; r < R; ++r) q[r] = 0.0f;
#pragma unroll 2
        for (int f = 0; f < d4; ++f) {
            f32x4 y;
            if constexpr (VW == 4) { // d is a multiple of 4
                y = *reinterpret_cast<const f32x4 *>(cj + 4 * f);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float z = cj[4 * f + e < a.d ? 4 * f + e : 0];
                    y[e] = 4 * f + e < a.d ? z : 0.0f;
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const f32x4 x = *reinterpret_cast<const f32x4 *>(&xs[f][r][0]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float diff = x[e] - y[e];
                    q[r] = fmaf(diff, diff, q[r]);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) farthest = max(farthest, __float_as_uint(q[r]));
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float x = fminf(a.s2 * q[r], a.most);
            float p;
            if constexpr (KIND == KNM_KERNEL_GAUSSIAN) p = __builtin_amdgcn_exp2f(-x);
            else p = radial_from_exponent<KIND>(-x);
#pragma unroll
            for (int c = 0; c < TP; ++c) sum[r][c] = fmaf(p, v[c], sum[r][c]);
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < TP; ++c) {
            float s = sum[r][c];
#pragma unroll
            for (int w = 32; w > 0; w >>= 1) s += __shfl_xor(s, w);
            if (lane == 0) red[wave][r * TP + c] = s;
        }
    __syncthreads();
    if (tid < R * TP) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) s += (double)red[w][tid];
        const int64_t row = row0 + tid / TP;
        const int c = tid % TP;
        if (row < a.n && c < a.t) {
            if (a.part != nullptr) a.part[((int64_t)blockIdx.y * a.n + row) * a.t + c] = s;
            else a.out[row * a.t + c] = (float)s;
        }
    }
    if (a.range_count != nullptr && __syncthreads_or(!(a.s2 * __uint_as_float(farthest) <= kNormMax / 9.0f))) count_out_of_range<R>(a, row0, j0, j1);
}

int columns(int t) { return t == 1 ? 1 : t == 2 ? 2 : t <= 4 ? 4 : t <= 8 ? 8 : 16; }
int rows(int t) { return t <= 4 ? 4 : t <= 8 ? 2 : 1; }

} // namespace

// workgroups along the centres: whole chunks, or fewer centres each where the rows alone leave compute units without one
int direct_chunks(int64_t n, int64_t M, int t)
{
    const int64_t groups = (n + rows(t) - 1) / rows(t);
    const int64_t most = (M + kThreads - 1) / kThreads;
    int64_t chunks = (M + kChunk - 1) / kChunk;
    if (M > 2048 && chunks * groups < 256) chunks = (256 + groups - 1) / groups;
    if (chunks > most) chunks = most;
    const int64_t len = ((M + chunks - 1) / chunks + kThreads - 1) / kThreads * kThreads;
    return (int)((M + len - 1) / len);
}

// Where this launch (and the merge of a split row) takes less time than the four or more of the engines.  Estimates in us, fitted at d = 2
// to 128, t = 1 to 16, n = 1 to 1000000, M = 1 to 50000, four kernels and both cross terms (1625 shapes).  What the differences of the values
// take: 5 + 0.03 to 0.07 ps per value and operation (twice that where rows cannot be read 16 bytes at a time, more where several columns leave
// fewer rows per workgroup), the engines 20 + 0.2 ps per value.  What a workgroup takes, however few its centres are: one pass after
// the other over 256 of them, each a chain of loads, and 1 ns per group of rows with 1 column, 3.6 from 3 on, for the sums over its threads (16
// sums of 6 steps through LDS).  The engines: 28 and more with 8 columns (the column maxima, and one workgroup per 128 rows of few), in the
// fp32 mode more with many features.  Measured from Python (9 us at least), engines and this launch: n = 200, M = 1000, d = 8, 1 column 21.4
// and 9.1, n = 1000, M = 4000, d = 28 25.6 and 20.3, n = 20000, M = 1000, d = 8 25.1 and 16.8, n = 5000, M = 300, d = 8, 8 columns 31.9
// and 19.3; beyond the line n = 1000, M = 4000, d = 44 27.4 and 33.4, n = 20000, M = 300, d = 8, 3 columns 22.3 and 27.6, n = 100000, M = 100, d =
// 8 22.3 and 34.7, n = 1000000, M = 1, d = 8 82.5 and 315, with 16 columns 142 and 4290.
bool direct_pays(int64_t n, int64_t M, int d, int t, bool wide, int cross_term)
{
    if (d > kMaxD || t > 16 || n > 1000000 || M > 1000000) return false;
    const double values = 1.0e-6 * (double)n * (double)M, ops = 2.0 * d + 8.0 + 2.0 * t;
    const double ps = (0.03 + 0.0003 * d) * (wide ? 1.0 : 2.0) * (t <= 2 ? 1.0 : t <= 4 ? 1.3 : t <= 8 ? 2.5 : 5.0);
    const int chunks = direct_chunks(n, M, t), sums = rows(t) * columns(t), quads = (d + 3) / 4;
    const double least = 5.0 + (chunks > 1 ? 4.0 : 0.0);
    const double groups = (double)((n + rows(t) - 1) / rows(t)) * (double)chunks;
    const double passes = (double)(((M + chunks - 1) / chunks + kThreads - 1) / kThreads);
    const double pass = (columns(t) > 4 ? 0.05 * (columns(t) - 4) : 0.0) +
                        (sums <= 4 ? 0.02 : sums <= 8 ? 0.13 : 0.15) * (t > 4 ? 0.5 : 1.0) * (wide ? 1.0 : 3.0) * quads;
    const double workgroups = passes * pass + 1.0e-3 * groups * (0.2 + 0.21 * sums + 0.005 * quads) + (columns(t) == 16 ? 8.0 * values : 0.0);
    const double engines = cross_term != KNM_CROSS_F16X3 ? 20.0 + 0.12 * d : t >= 8 ? 28.0 + 0.011 * (double)(M < 4000 ? M : 4000) : 20.0;
    return least + values * ops * ps < 0.95 * (20.0 + 0.2 * values) && least + workgroups < 0.95 * (engines + 0.2 * values);
}
// (squares of differences and of sigma have to stay within fp32; the engines scale before they square)
bool direct_takes(float sigma) { return sigma >= 1.0e-15f && sigma <= 1.0e15f; }
bool direct_wide(const float *C, int64_t ldc, int d) { return d % 4 == 0 && ldc % 4 == 0 && (reinterpret_cast<uintptr_t>(C) & 15) == 0; }

hipError_t launch_direct(const float *X, int64_t n, int64_t ldx, const float *C, int64_t M, int64_t ldc, int d, float sigma, int kind,
                         const float *V, int t, float *out, double *part, unsigned int *range_count, float inv2s2, hipStream_t stream)
{
    if (n <= 0 || M <= 0 || d <= 0 || d > kMaxD || t <= 0 || t > 16 || kind < KNM_KERNEL_GAUSSIAN || kind > KNM_KERNEL_MATERN52) return hipErrorInvalidValue;
    const int chunks = direct_chunks(n, M, t);
    if ((chunks > 1) != (part != nullptr) || chunks > 65535) return hipErrorInvalidValue;
    DirectArgs a;
    a.X = X; a.n = n; a.ldx = ldx;
    a.C = C; a.M = M; a.ldc = ldc;
    a.V = V; a.t = t;
    a.d = d;
    a.s2 = kLog2e / (2.0f * sigma * sigma);
    a.chunk = (int)(((M + chunks - 1) / chunks + kThreads - 1) / kThreads * kThreads);
    a.out = out;
    a.part = part;
    a.range_count = range_count;
    a.inv2s2 = inv2s2;
    // 2^-1e30 and 2^-1e15 are 0: a point with a feature that is not finite or too large to square has the value 0, as with the engines, which
    // clamp it, and does not make a NaN of every other point's result (a Matern kernel's 0 times infinity).  Where nothing is clamped, kernels
    // of r carry a NaN on.
    a.most = kind == KNM_KERNEL_GAUSSIAN || range_count != nullptr ? 1.0e30f : std::numeric_limits<float>::quiet_NaN();
    const int64_t groups = (n + rows(t) - 1) / rows(t);
    if (groups > 0x7fffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)groups, (unsigned)chunks);
    const bool wide = direct_wide(C, ldc, d);
    auto launch = [&](auto kd) {
        constexpr int K = decltype(kd)::value;
        auto go = [&](auto r, auto tp) {
            if (wide) hipLaunchKernelGGL((direct_kernel<K, decltype(r)::value, decltype(tp)::value, 4>), grid, dim3(kThreads), 0, stream, a);
            else hipLaunchKernelGGL((direct_kernel<K, decltype(r)::value, decltype(tp)::value, 1>), grid, dim3(kThreads), 0, stream, a);
        };
        switch (columns(t)) {
        case 1: go(std::integral_constant<int, 4>{}, std::integral_constant<int, 1>{}); break;
        case 2: go(std::integral_constant<int, 4>{}, std::integral_constant<int, 2>{}); break;
        case 4: go(std::integral_constant<int, 4>{}, std::integral_constant<int, 4>{}); break;
        case 8: go(std::integral_constant<int, 2>{}, std::integral_constant<int, 8>{}); break;
        default: go(std::integral_constant<int, 1>{}, std::integral_constant<int, 16>{}); break;
        }
    };
    switch (kind) {
    case KNM_KERNEL_LAPLACIAN: launch(std::integral_constant<int, KNM_KERNEL_LAPLACIAN>{}); break;
    case KNM_KERNEL_MATERN32: launch(std::integral_constant<int, KNM_KERNEL_MATERN32>{}); break;
    case KNM_KERNEL_MATERN52: launch(std::integral_constant<int, KNM_KERNEL_MATERN52>{}); break;
    default: launch(std::integral_constant<int, KNM_KERNEL_GAUSSIAN>{}); break;
    }
    return hipGetLastError();
}

} // namespace knm
