// Sums over kept kernel values with many columns: out[i, c] = sum_j K[i, j] vec[j, c] (see knm_internal.h for the layout of K), up to
// 160 columns per launch on the f16 matrix cores.
//
// The arithmetic is that of the K-loop engine's reduction on the matrix cores: values times 2^14 in two halves, the vectors' halves from
// their packed image (launch_vector_image), three products, fp32 sums over a chunk.  A wavefront has 32 of the points that the result
// runs over, and a sum of 32 columns per group; a value is read once for all columns.  A lane of the product's second operand holds 8 values of one such
// point: over the stream points two units of 4 rows, over the fixed ones 8 values of as many units.  Values and vectors come by loads that
// write LDS directly, two stages of 32 points ahead of their use; a lane fetches the unit whose place in LDS is its own, so that a block's units
// lie where reading it over the stream has no bank conflicts, and reading it over the fixed points 7 % of the clocks in them.
// Bound by the matrix cores (busy half of the clocks, at 1.6 to 1.9 GHz) and the values' bandwidth together, 120000 x 20000 values, 144 columns:
// 2.9 ms over the centres, 2.8 over the rows (3.3 TB/s); with the values in registers a stage ahead 3.0 and 3.2; vectors read where they are used 3.7
// and 3.0; values through the caches 3.2 and 3.0.
#include <type_traits>

#include "knm_internal.h"
#include "knm_operands.h"

namespace knm {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 512; // eight wavefronts, one workgroup per CU
constexpr int kWaves = kThreads / 64;
constexpr int kOut = 32 * kWaves;  // points of the result of a workgroup
constexpr int kRing = 3;           // stages of 32 points in LDS
constexpr int kBlockUnits = kKeptBlock / 4; // 16-byte units of a block of values, and of a stage's vectors per group of 32 columns: [K-step][plane][lane]
constexpr int kTileUnits = 4 * kBlockUnits; // of a group's vectors of a tile of 128 points in the image

struct ManyArgs {
    const float *values;
    int64_t n_s32;       // stream blocks per 32 fixed points
    int64_t out_blocks;  // blocks of 32 points of the result there are values for
    int64_t n_out;
    int64_t stages;      // of 32 points summed over, in all
    int64_t chunk;       // stages per chunk
    const f16x8 *vimg;
    const uint32_t *colmax;
    int t;               // columns of this launch
    float *part;         // part[chunk * part_stride + i * ldo + c]
    int64_t part_stride, ldo;
};

// Where unit (f, rq, y), rows 8 rq + 4 y ... + 3 of the stream for fixed point f, of a block lies in LDS: the 16 units of f = 0 .. 15
// or 16 .. 31 and the 16 of one value each (two f apart by 4, all rq and y) are in different banks.
__device__ __forceinline__ int turned(int f, int rq, int y)
{
    const int a0 = (f >> 2) & 1, a1 = (f >> 3) & 1, a2 = f >> 4, c0 = f & 1, c1 = (f >> 1) & 1, x0 = rq & 1, x1 = rq >> 1;
    return (a2 * 8 + x0 * 4 + x1 * 2 + y) * 16 + (a0 | (a1 ^ x0) << 1 | (c0 ^ x1) << 2 | (c1 ^ y) << 3);
}
// the unit that lies there, by its place in memory
__device__ __forceinline__ int unit_at(int place)
{
    const int y = (place >> 4) & 1, x1 = (place >> 5) & 1, x0 = (place >> 6) & 1, a2 = place >> 7;
    const int a0 = place & 1, a1 = ((place >> 1) & 1) ^ x0, c0 = ((place >> 2) & 1) ^ x1, c1 = ((place >> 3) & 1) ^ y;
    return kept_unit((a2 << 4) | (a1 << 3) | (a0 << 2) | (c1 << 1) | c0, y) + 8 * (2 * x1 + x0);
}

template <int G, bool OVER_STREAM>
__global__ __launch_bounds__(kThreads, 2) void kept_many_kernel(ManyArgs a)
{
    extern __shared__ f16x8 lds[]; // [kRing][blocks of the wavefronts, groups of vectors][kBlockUnits]
    constexpr int kPieces = kWaves + G;
    const int tid = threadIdx.x, lane = tid & 63, l31 = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t o = (int64_t)blockIdx.x * kWaves + wave; // block of the result
    const int64_t ob = o < a.out_blocks ? o : 0;
    const int64_t first = (int64_t)blockIdx.y * a.chunk;
    const int stages = (int)(first + a.chunk <= a.stages ? a.chunk : a.stages - first);
    const int64_t step = OVER_STREAM ? kKeptBlock : a.n_s32 * kKeptBlock; // from a block summed over to the next
    const float *const src = a.values + (OVER_STREAM ? ob * a.n_s32 : ob) * kKeptBlock + first * step;

    // A wavefront's loads of a stage: the four of its own block, and every eighth of the 4 G of the vectors, 1 KB each.
    constexpr int kVecLoads = 4 * G / kWaves, kVecRest = 4 * G % kWaves; // (the first kVecRest wavefronts one more)
    unsigned from[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) from[k] = (unsigned)unit_at(k * 64 + lane) * 16u;
    const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) f16x8 *)&lds[0]);
    // (one wait state between a scalar write of M0 and the load that reads it; the values, which are read once, past the caches that hold the vectors)
#define KNM_FETCH(hint)                                                                                                                      \
    asm volatile("s_mov_b32 %[keep], m0\n\ts_mov_b32 m0, %[l]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[o], %[b]" hint "\n\ts_mov_b32 m0, %[keep]" \
                 : [keep] "=&s"(keep)                                                                                                        \
                 : [l] "s"(__builtin_amdgcn_readfirstlane(to)), [o] "v"(offset), [b] "s"(uniform_pointer(static_cast<const char *>(base)))    \
                 : "memory")
    auto fetch_value = [&](const void *base, unsigned offset, unsigned to) {
        unsigned keep;
        KNM_FETCH(" nt");
    };
    auto fetch = [&](const void *base, unsigned offset, unsigned to) {
        unsigned keep;
        KNM_FETCH("");
    };
#undef KNM_FETCH
    auto issue = [&](int st, int slot) {
        const unsigned to = lds0 + (unsigned)(slot * kPieces * kBlockUnits * 16);
        const float *const block = src + (int64_t)st * step;
#pragma unroll
        for (int k = 0; k < 4; ++k) fetch_value(block, from[k], to + (unsigned)(wave * kBlockUnits + k * 64) * 16u);
        const int64_t stage = first + st;
        const f16x8 *const vec = a.vimg + (stage >> 2) * (G * kTileUnits) + (stage & 3) * kBlockUnits;
#pragma unroll
        for (int i = 0; i <= kVecLoads; ++i) {
            const int piece = wave + kWaves * i; // of 64 units: piece % 4 of group piece / 4
            if (i < kVecLoads || wave < kVecRest)
                fetch(vec + (piece >> 2) * kTileUnits + (piece & 3) * 64, (unsigned)lane * 16u, to + (unsigned)(kWaves * kBlockUnits + piece * 64) * 16u);
        }
    };

    f32x16 acc[G];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[g][r] = 0.0f;

    constexpr float kScale = 16384.0f; // the halves then resolve values down to 4e-9
    auto work = [&](int slot) {
        const f16x8 *const stage = lds + slot * kPieces * kBlockUnits;
        const float *const block = reinterpret_cast<const float *>(stage + wave * kBlockUnits);
        const f16x8 *const vec = stage + kWaves * kBlockUnits + lane;
        float x[16]; // by K-slot: point 8 (k / 4) + 4 h + k % 4 of the stage
        if constexpr (OVER_STREAM) {
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                const f32x4 v = *reinterpret_cast<const f32x4 *>(block + turned(l31, rq, h) * 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[4 * rq + e] = v[e];
            }
        } else {
#pragma unroll
            for (int k = 0; k < 16; ++k) x[k] = block[turned(8 * (k >> 2) + 4 * h + (k & 3), l31 >> 3, (l31 >> 2) & 1) * 4 + (l31 & 3)];
        }
        // Group u = (K-step, group of columns): the vectors of the next one are read, and a part of the next K-step's values
        // converted, before and between this one's products.
        u32x4 ph[2], pl[2];
        auto convert = [&](int q, int e) {
            const float p0 = kScale * x[8 * q + e], p1 = kScale * x[8 * q + e + 1];
            const f16x2 h2 = __builtin_amdgcn_cvt_pkrtz(p0, p1);
            const f16x2 l2 = __builtin_amdgcn_cvt_pkrtz(p0 - (float)h2[0], p1 - (float)h2[1]);
            ph[q][e / 2] = __builtin_bit_cast(uint32_t, h2);
            pl[q][e / 2] = __builtin_bit_cast(uint32_t, l2);
        };
        f16x8 vh[2], vl[2];
        auto read = [&](int u) {
            vh[u & 1] = vec[(u % G) * kBlockUnits + (u / G) * 128];
            vl[u & 1] = vec[(u % G) * kBlockUnits + (u / G) * 128 + 64];
        };
        read(0);
#pragma unroll
        for (int e = 0; e < 8; e += 2) convert(0, e);
#pragma unroll
        for (int u = 0; u < 2 * G; ++u) {
            const int q = u / G, g = u % G;
            if (u + 1 < 2 * G) read(u + 1);
            __builtin_amdgcn_sched_barrier(0);
            const f16x8 bh = __builtin_bit_cast(f16x8, ph[q]), bl = __builtin_bit_cast(f16x8, pl[q]);
            acc[g] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vh[u & 1], bh, acc[g], 0, 0, 0);
            acc[g] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vh[u & 1], bl, acc[g], 0, 0, 0);
            if (q == 0)
#pragma unroll
                for (int e = 8 * g / G / 2 * 2; e < 8 * (g + 1) / G / 2 * 2; e += 2) convert(1, e);
            acc[g] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vl[u & 1], bh, acc[g], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    if (stages > 0) issue(0, 0);
    if (stages > 1) issue(1, 1);
    int slot = 0;
    for (int st = 0; st < stages; ++st) {
        // this stage's loads have landed when no more are under way than the next one's
        if (st + 1 >= stages) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        else if (wave < kVecRest) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 + kVecLoads + 1) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 + kVecLoads) : "memory");
        __syncthreads(); // everyone's have, and the slot of the stage before this one is free
        if (st + 2 < stages) issue(st + 2, slot == 0 ? kRing - 1 : slot - 1);
        __builtin_amdgcn_sched_barrier(0);
        work(slot);
        slot = slot == kRing - 1 ? 0 : slot + 1;
    }

    // register r of a lane, group g: column 32 g + 8 (r / 4) + 4 h + r % 4 of point lane % 32
    const int64_t i = o * 32 + l31;
    if (o >= a.out_blocks || i >= a.n_out) return;
    float *const out = a.part + (int64_t)blockIdx.y * a.part_stride + i * a.ldo;
    const bool whole = a.t % 4 == 0 && a.ldo % 4 == 0 && a.part_stride % 4 == 0 && (reinterpret_cast<uintptr_t>(a.part) & 15) == 0;
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
            const int c = 32 * g + 8 * rq + 4 * h;
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (acc[g][4 * rq + e] * (1.0f / kScale)) * column_scale(a.colmax[c + e], true);
            if (whole) {
                if (c < a.t) *reinterpret_cast<f32x4 *>(out + c) = v;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (c + e < a.t) out[c + e] = v[e];
            }
        }
}

} // namespace

int kept_many_max_t() { return 160; }

hipError_t launch_kept_many(const KeptManyArgs &k, hipStream_t stream)
{
    if (k.nF <= 0 || k.nS <= 0 || k.t <= 0 || k.t > kept_many_max_t() || k.chunk_len <= 0 || k.chunk_len % 128 != 0) return hipErrorInvalidValue;
    ManyArgs a;
    a.values = k.values;
    a.n_s32 = kept_stream_blocks(k.nS);
    a.out_blocks = k.over_stream ? kept_rows(k.nF) / 32 : a.n_s32;
    a.n_out = k.over_stream ? k.nF : k.nS;
    const int64_t n_in = k.over_stream ? k.nS : k.nF;
    a.stages = (n_in + 31) / 32;
    a.chunk = k.chunk_len / 32;
    a.vimg = static_cast<const f16x8 *>(k.vimg);
    a.colmax = k.colmax;
    a.t = k.t;
    a.part = k.part;
    a.part_stride = k.part_stride;
    a.ldo = k.ldo;
    const int64_t chunks = (a.stages + a.chunk - 1) / a.chunk, wgs = (a.n_out + kOut - 1) / kOut;
    if (chunks > 65535 || wgs > 0x7fffff || a.chunk > 1 << 20) return hipErrorInvalidValue;
    const dim3 grid((unsigned)wgs, (unsigned)chunks);
    auto launch = [&](auto groups) {
        constexpr int G = decltype(groups)::value;
        const size_t bytes = (size_t)kRing * (kWaves + G) * kBlockUnits * sizeof(f16x8);
        auto *kernel = k.over_stream ? kept_many_kernel<G, true> : kept_many_kernel<G, false>;
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, grid, dim3(kThreads), bytes, stream, a);
        return hipGetLastError();
    };
    if (k.t <= 32) return launch(std::integral_constant<int, 1>{});
    if (k.t <= 64) return launch(std::integral_constant<int, 2>{});
    if (k.t <= 128) return launch(std::integral_constant<int, 4>{});
    return launch(std::integral_constant<int, 5>{});
}

} // namespace knm
