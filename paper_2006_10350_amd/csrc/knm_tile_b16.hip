// Gaussian-kernel tile engine with the fp32 cross term on the bf16 matrix cores:
//     out[f] = sum_s k(F_f, S_s) vec[s]          (KNM_CROSS_F32, d <= 14, one column per launch)
//
// Same computation as knm_tile.hip, whose fp32 MFMA shares the vector ALU's issue with the exp/FMA work that finishes every
// kernel value, so that its time is that of both.  A bf16 MFMA has 16 times the rate and runs beside the vector ALU.
// bf16 has the exponents of fp32 and 8 bits of its 24, so a number is the sum of three of them, rounded to nearest each
// time, whatever its magnitude and to 2^-27 of it: z = z1 + z2 + z3, |z2| <= 2^-9 |z|, |z3| <= 2^-18 |z|, and nothing has to be clamped.  Of the nine
// products of two such sums the six with
//     f1 x1, f1 x2, f2 x1, f2 x2, f1 x3, f3 x1
// are formed (exactly, and added in fp32); f2 x3, f3 x2 and f3 x3 are below 2^-26 of f x together, a quarter of the
// rounding of an fp32 number, and of either sign.  The exponent log2 k = <zf, zx> - |zf|^2 / 2 - |zx|^2 / 2 of z = x sqrt(log2 e) / sigma takes 6 contraction slots per
// feature and 8 for the two norm terms, 16 slots to an MFMA: 4 MFMAs of 32 cycles per 32 x 32 tile at d = 9, where fp32 has 7 of 64.
// 1M x 20k, d = 9: 11.7 -> 5.1 ms per product, d = 4 6.7 -> 3.8, d = 14 13.5 -> 6.8.  Error against 64 bits relative to that of the fp32 MFMA engine, over
// d = 1 to 14, normal rows and half whole-valued, half skewed ones, three sigmas, vectors of either sign and positive ones, 120000 x 3000 and 40000 x 9000: W
// 0.56 and U 0.34 (geometric means), at most 1.05 (W, d = 5, 40000 x 9000) and 1.04 (U, d = 12, 2.6e-8: the rounding of the result).
// Bound by the exp/FMA work of the vector ALU and the matrix cores beside it, which overlap in part: 256 clocks of MFMA and 384 of
// exp/FMA per pair of tiles take 630 at d = 9.
//
// Layout and schedule are those of knm_tile_f16.hip: the stream points are packed once per sweep (or fit) into an image laid out as
// the LDS stage, per 32-point tile [MFMA][lane] units of 16 bytes; loads that write LDS directly bring a stage ahead of its
// use; the finish of a tile runs behind the MFMAs of the next.
#include <type_traits>

#include "knm_internal.h"
#include "knm_operands.h"

namespace knm {
namespace {

typedef uint32_t unit_t __attribute__((ext_vector_type(4))); // 8 bf16 numbers

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kSlots = 6;     // contraction slots per feature
constexpr int kNormSlots = 8; // and for the two norm terms
constexpr int kStage = 128; // stream points per LDS stage, as in knm_tile.hip
constexpr int kTilesPerStage = kStage / 32;
constexpr int waves_of(int nm) { return nm <= 4 ? 3 : 2; } // wavefronts per SIMD, workgroups per CU
// MFMAs of a tile: 16 slots each; and the features that fit so many
constexpr int mfmas_of(int d) { return d <= 4 ? 2 : (kSlots * d + kNormSlots + 15) / 16; }
constexpr int features_of(int nm) { return (16 * nm - kNormSlots) / kSlots; }
// The large terms, f1 x1 and part 1 of both norms, fit one MFMA up to 14 features.  From 15 on they take two, and what the first of these cuts off the second
// does not bring back: errors of up to 4.8 times those of the fp32 engine (d = 16, skewed rows, half the usual sigma).  (9 to 12.7 ms in place of 15.5
// to 20 at d = 20 to 28, 1M x 20k, but for that.)
constexpr int kMaxD = 14;
static_assert(features_of(mfmas_of(kMaxD)) + 2 <= 16, "the large terms of a sum in one instruction");

// bits of x rounded to bf16; x becomes the remainder
template <typename T> __device__ __forceinline__ uint32_t take_bf16(T &x)
{
    const __bf16 z = (__bf16)(float)x;
    x -= (T)(float)z;
    return __builtin_bit_cast(unsigned short, z);
}

// What slot s holds: the products from the least to the largest, f1 x3, f3 x1, f2 x2, parts 2 to 4 of the norm terms, f1 x2, f2 x1, f1 x1, part 1 of the
// norm terms, behind the zeros that fill the first MFMA; up to 9 features in the opposite order.  The matrix cores cut off what lies below the last bit of
// the largest term of a sum, always to the same side.  With the large terms last that happens once, but at their magnitude, and what it cuts off
// is the same for many pairs: U, which sums them twice, had 1.2 times the error of the fp32 engine on positive vectors at d = 2 and 1.15 at d = 6.  With the large terms
// first they have cancelled before the others come in, and every further MFMA cuts at the magnitude of the exponent alone: 0.42 and 0.40 times;
// but W was up to 1.18 times that engine's from 12 features on, five or six MFMAs, where the first order has 0.52 to 0.82 and U at most
// 0.6.  (Feature by feature, all six products of one side by side: W 1.07 times in place of 0.84 over all d.)
struct Slot {
    int feature = -1, part = 0; // part of that feature
    int norm = -1;              // or part of the norm term, 0 to 3, of this side
    bool one = false;           // or 1, for a part of the other side's
};
template <bool FIXED, int NM> constexpr Slot slot_at(int s)
{
    constexpr int D = features_of(NM);
    Slot r;
    s = NM <= 4 ? kSlots * D + kNormSlots - 1 - s : s - (16 * NM - kSlots * D - kNormSlots);
    if (s < 0) return r;
    int n = -1; // part of the fixed (0 to 3) or stream side's (4 to 7) norm term
    if (s < 3 * D) {
        r.feature = s % D;
        r.part = s / D == 2 ? 1 : (s / D == 1) == FIXED ? 2 : 0;
    } else if ((s -= 3 * D) < 6) {
        n = s < 3 ? s + 1 : s + 2;
    } else if ((s -= 6) < 3 * D) {
        r.feature = s % D;
        r.part = s / D == 2 ? 0 : (s / D == 1) == FIXED ? 1 : 0;
    } else {
        n = 4 * (s - 3 * D);
    }
    if (n >= 0 && (n < 4) == FIXED) r.norm = n & 3;
    else if (n >= 0) r.one = true;
    return r;
}

// The slots of half-wave h of a point: 8 of each MFMA.  Features z = gamma (p - mu) to 2^-33, of which the parts are taken, the same on both sides; norm
// term -|z|^2 / 2 of the sums of the parts in fp64, four parts of it (32 bits): what is left of the exponent of two coincident points is what
// the products leave out.  (Rounded to fp32 before, whole-valued features were off by the same amount in many rows: errors of U on skewed and whole-valued
// rows up to 1.4 times those of the fp32 engine at d = 13.)  gamma in two fp32 numbers and fp32 fused multiply-adds give what fp64 arithmetic gives here, in
// less time for the workgroups of small products (120000 x 3000, d = 9: 156 -> 145 us).
template <bool FIXED, int NM>
__device__ __forceinline__ void make_units(const float *__restrict__ p, const float *__restrict__ mu, int d, double gamma, bool valid, int h,
                                           unit_t (&units)[NM])
{
    constexpr int D = features_of(NM);
    float x[D];
    load_features<D, 1>(p, mu, true, 0, d, valid, x);
    const float gamma_hi = (float)gamma, gamma_lo = (float)(gamma - (double)gamma_hi);
    uint32_t part[D][3], norm_part[4];
    double norm = 0.0;
#pragma unroll
    for (int k = 0; k < D; ++k) {
        const float z1 = (float)(__bf16)(gamma_hi * x[k]);
        const float after = fmaf(gamma_lo, x[k], fmaf(gamma_hi, x[k], -z1)); // z - z1, to 2^-33 of z
        float rest = after;
        part[k][0] = __builtin_bit_cast(uint32_t, z1) >> 16;
        part[k][1] = take_bf16(rest);
        part[k][2] = take_bf16(rest);
        const double z = (double)z1 + (double)(after - rest); // the parts' sum
        norm = fma(-0.5 * z, z, norm);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) norm_part[q] = take_bf16(norm);
    const uint32_t one = valid ? 0x3f80u : 0u;
    auto value = [&](const Slot &s) { return s.feature >= 0 ? part[s.feature][s.part] : s.norm >= 0 ? norm_part[s.norm] : s.one ? one : 0u; };
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int s = 16 * m + 2 * e;
            const uint32_t lo = value(slot_at<FIXED, NM>(s)) | value(slot_at<FIXED, NM>(s + 1)) << 16;
            const uint32_t hi = value(slot_at<FIXED, NM>(s + 8)) | value(slot_at<FIXED, NM>(s + 9)) << 16;
            units[m][e] = h ? hi : lo;
        }
}

// Image of the stream points [row0, row0 + rows), rows a multiple of 32 (those beyond nS are zeros).
template <int NM>
__global__ __launch_bounds__(kThreads) void pack_stream_b16_kernel(const float *__restrict__ S, int64_t nS, int64_t lds,
                                                                  const float *__restrict__ mu, int d, double gamma, int64_t row0,
                                                                  int64_t rows, unit_t *__restrict__ packed)
{
    const int h = (threadIdx.x >> 5) & 1, prow = threadIdx.x & 31;
    const int64_t tile = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (tile * 32 >= rows) return;
    const int64_t idx = row0 + tile * 32 + prow;
    const bool valid = idx < nS;
    unit_t units[NM];
    make_units<false, NM>(S + (valid ? idx : 0) * lds, mu, d, gamma, valid, h, units);
#pragma unroll
    for (int m = 0; m < NM; ++m) packed[(tile * NM + m) * 64 + h * 32 + prow] = units[m];
}

template <bool FIRST>
__device__ __forceinline__ void mfma_step(f32x16 &acc, const unit_t &a, const unit_t &b)
{
    if constexpr (FIRST) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(a), "v"(b));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}

// s_r += min(max(2^x_r, 0), 1) vl for entries R0 .. R0 + G - 1 of a finished tile.  One volatile statement per instruction, in program order; an
// exponential is never read by the instruction right after it.
template <int G, int R0>
__device__ __forceinline__ void finish_group(const f32x16 &pa, float vl, float (&s)[16])
{
    float p[G];
#pragma unroll
    for (int i = 0; i < G; ++i) asm volatile("v_exp_f32_e64 %0, %1 clamp" : "=v"(p[i]) : "v"(pa[R0 + i]));
    if constexpr (G == 1) asm volatile("s_nop 0");
#pragma unroll
    for (int i = 0; i < G; ++i) asm volatile("v_fmac_f32_e32 %0, %1, %2" : "+v"(s[R0 + i]) : "v"(p[i]), "v"(vl));
}

// The MFMAs of one fixed block on one stream tile, with the finish of the same block's previous tile (`pa`, weight `vl_prev`)
// spread behind them; RELOAD: operand I of the next tile (at next[64 I]) takes the place of this one's once it has been used.
template <int NM, bool RELOAD, int I = 0>
__device__ __forceinline__ void block_tile(f32x16 &acc, const unit_t (&f)[NM], unit_t (&b)[NM], const f32x16 &pa, float vl_prev,
                                           float (&s)[16], const unit_t *next)
{
    if constexpr (I < NM) {
        constexpr int R0 = 16 * I / NM, G = 16 * (I + 1) / NM - R0;
        mfma_step<I == 0>(acc, f[I], b[I]);
        finish_group<G, R0>(pa, vl_prev, s);
        if constexpr (RELOAD) {
            __builtin_amdgcn_sched_barrier(0);
            b[I] = next[64 * I];
            __builtin_amdgcn_sched_barrier(0);
        }
        block_tile<NM, RELOAD, I + 1>(acc, f, b, pa, vl_prev, s, next);
    }
}

// UPT units of 16 bytes per thread from `from` to the LDS address `lds` of the wavefront (the same in every lane): unit k of the
// thread at from[k kThreads + thread].  Counted by vmcnt; the caller waits.
template <int UPT>
__device__ __forceinline__ void stage_units(const unit_t *from, unsigned lds, unsigned offset)
{
#pragma unroll
    for (int k = 0; k < UPT; ++k) {
        unsigned keep;
        // (one wait state between a scalar write of M0 and the load that reads it)
        asm volatile("s_mov_b32 %[keep], m0\n\ts_mov_b32 m0, %[l]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[o], %[b]\n\ts_mov_b32 m0, %[keep]"
                     : [keep] "=&s"(keep)
                     : [l] "s"(lds + 0x1000u * k), [o] "v"(offset), [b] "s"(from + k * kThreads)
                     : "memory");
    }
}

// `packed` is the image of the stream chunks [chunk0, chunk0 + n_chunks).  Workgroups are numbered as those of
// gauss_sweep_f16_kernel: the first 8 floor(n_chunks / 8) chunks run on one XCD each.
template <int NM>
__global__ __launch_bounds__(kThreads, waves_of(NM)) void gauss_sweep_b16_kernel(SweepArgs a, double gamma, const unit_t *__restrict__ packed,
                                                                      int64_t chunk0, int n_fblocks, int n_chunks)
{
    int64_t fblock, chunk_local;
    const int grouped = n_chunks & ~7; // chunks that are dealt to one XCD each
    const unsigned blocks = (unsigned)n_fblocks; // (the grid's size fits 31 bits)
    if (blockIdx.x < (unsigned)grouped * blocks) {
        const unsigned slot = blockIdx.x >> 3;
        chunk_local = (slot / blocks) * 8 + (blockIdx.x & 7);
        fblock = slot % blocks;
    } else {
        const unsigned rest = blockIdx.x - (unsigned)grouped * blocks;
        fblock = rest % blocks;
        chunk_local = grouped + rest / blocks;
    }

    constexpr int UPS = kTilesPerStage * NM * 64; // units per stage
    constexpr int UPT = UPS / kThreads;
    __shared__ unit_t img[2][kTilesPerStage][NM][64]; // [buffer][tile][MFMA][lane]
    __shared__ float vv[2][kStage];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int row = lane & 31;
    const int h = lane >> 5;

    const int64_t fixed0 = (fblock * kWaves + wave) * 64;
    float sum[2][16];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int r = 0; r < 16; ++r) sum[rb][r] = 0.0f;

    const int64_t chunk = chunk0 + chunk_local;
    const int64_t chunk_begin = chunk * a.chunk_len;
    int64_t chunk_end = chunk_begin + a.chunk_len;
    if (chunk_end > a.nS) chunk_end = a.nS;
    const int n_stages = (int)((chunk_end - chunk_begin + kStage - 1) / kStage);
    const unit_t *const src = packed + (chunk_local * a.chunk_len / kStage) * UPS;
    const unsigned lds_wave = __builtin_amdgcn_readfirstlane(
        (unsigned)(uintptr_t)(__attribute__((address_space(3))) unit_t *)&img[0][0][0][0] + (unsigned)wave * 1024u);
    auto issue = [&](int stage, int buf) {
        stage_units<UPT>(uniform_pointer(src + (int64_t)stage * UPS),
                         __builtin_amdgcn_readfirstlane(lds_wave + (unsigned)buf * (unsigned)(UPS * 16)), (unsigned)tid * 16u);
    };
    float vs = 0.0f;
    auto fetch = [&](int stage) {
        const int64_t idx = chunk_begin + (int64_t)stage * kStage + (tid & (kStage - 1));
        const bool valid = idx < chunk_end;
        const int64_t vi = valid ? idx : 0;
        const float vraw = a.vec[vi * a.ldv];
        const float wraw = (a.wgt != nullptr) ? a.wgt[vi] : 1.0f;
        vs = valid ? vraw * wraw : 0.0f;
    };

    if (n_stages > 0) {
        issue(0, 0);
        fetch(0);
    }

    // fixed operand: 2 blocks of 32 points per wavefront, in registers
    unit_t f[2][NM];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
        const int64_t idx = fixed0 + rb * 32 + row;
        const bool valid = idx < a.nF;
        const float *p = a.F + (valid ? idx : 0) * a.ldf;
        make_units<true, NM>(p, a.mu, a.d, gamma, valid, h, f[rb]);
    }

    // accumulators of the tile in flight and of the tile being finished
    f32x16 accA[2], accB[2];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int r = 0; r < 16; ++r) { accA[rb][r] = 0.0f; accB[rb][r] = 0.0f; }
    float vl_prev = 0.0f; // zero weight: the first "previous tile" contributes nothing

    for (int st = 0; st < n_stages; ++st) {
        const int buf = st & 1;
        if (tid < kStage) vv[buf][tid] = vs;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // this thread's share of the stage has landed
        __syncthreads();                                 // everyone's has, and the other buffer is free
        if (st + 1 < n_stages) {
            issue(st + 1, buf ^ 1);
            fetch(st + 1);
        }
        unit_t b[NM];
#pragma unroll
        for (int m = 0; m < NM; ++m) b[m] = img[buf][0][m][lane];
        float vl = vv[buf][row];
#pragma unroll
        for (int tile = 0; tile < kTilesPerStage; ++tile) {
            constexpr int kLast = kTilesPerStage - 1;
            const int to = tile < kLast ? tile + 1 : tile;
            const unit_t *next = &img[buf][to][0][lane];
            auto both = [&](f32x16 (&now)[2], const f32x16 (&before)[2]) {
                block_tile<NM, false>(now[0], f[0], b, before[0], vl_prev, sum[0], next);
                if (tile < kLast) block_tile<NM, true>(now[1], f[1], b, before[1], vl_prev, sum[1], next);
                else block_tile<NM, false>(now[1], f[1], b, before[1], vl_prev, sum[1], next);
            };
            if ((tile & 1) == 0) both(accA, accB);
            else both(accB, accA);
            vl_prev = vl;
            vl = vv[buf][to * 32 + row];
        }
    }
    // the last tile's accumulators (in set B); the wait states an MFMA result needs before ordinary code may read it are
    // explicit, because the compiler does not know that the inline assembly above contains MFMAs
    static_assert(kTilesPerStage % 2 == 0, "accumulator sets alternate per tile");
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 3" : "+v"(accB[0]), "+v"(accB[1]));
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            sum[rb][r] = fmaf(__builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(accB[rb][r]), 0.0f, 1.0f), vl_prev, sum[rb][r]);

    // reduce over the 32 stream lanes of each half-wave and store
    float *out = a.out + chunk * a.chunk_stride;
    const float total = half_wave_sums(sum);
    const int64_t idx = fixed0 + half_wave_point(row, h);
    if (idx < a.nF) out[idx * a.ldo] = total;
}

template <int NM>
hipError_t launch_nm(const SweepArgs &a, void *pack_buf, size_t pack_bytes, hipStream_t stream)
{
    const int64_t per_block = (int64_t)kWaves * 64;
    const int64_t blocks = (a.nF + per_block - 1) / per_block;
    // slab = whole chunks whose image fits the workspace
    const int64_t slab_chunks = a.simg != nullptr ? a.n_chunks : (int64_t)(pack_bytes / (size_t)(32 * NM)) / a.chunk_len;
    if (slab_chunks < 1) return hipErrorInvalidValue;
    const double gamma = sqrt(1.4426950408889634) / (double)a.sigma;
    unit_t *packed = static_cast<unit_t *>(a.simg != nullptr ? a.simg : pack_buf);
    for (int64_t c0 = 0; c0 < a.n_chunks; c0 += slab_chunks) {
        const int64_t nc = (a.n_chunks - c0 < slab_chunks) ? a.n_chunks - c0 : slab_chunks;
        const int64_t rows = nc * a.chunk_len, wgs = blocks * nc;
        if (wgs > 0x7fffffff || rows > (int64_t)1 << 36) return hipErrorInvalidValue;
        if (a.simg == nullptr || !a.simg_ready)
            hipLaunchKernelGGL((pack_stream_b16_kernel<NM>), dim3((unsigned)((rows + kThreads / 2 - 1) / (kThreads / 2))), dim3(kThreads), 0, stream, a.S,
                               a.nS, a.lds, a.mu, a.d, gamma, c0 * a.chunk_len, rows, packed);
        hipLaunchKernelGGL((gauss_sweep_b16_kernel<NM>), dim3((unsigned)wgs), dim3(kThreads), 0, stream, a, gamma, packed, c0, (int)blocks, (int)nc);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

} // namespace

int b16_workgroups_per_cu(int d) { return waves_of(mfmas_of(d)); }
// Whether a sweep over `entries` kernel values gains more than the launch that packs its stream points costs: 0.05 + 0.006 d ps per value
// against 7 us.  5003 x 501 35 -> 42 us, 60000 x 2000 124 -> 87 us per product at d = 9 with every sweep on this engine.
bool b16_pays(double entries, int d) { return d <= kMaxD && entries * (0.05 + 0.006 * d) > 7.0e6; }
size_t b16_pack_bytes_per_point(int d) { return (size_t)32 * mfmas_of(d); }

hipError_t launch_sweep_b16(const SweepArgs &a, void *pack_buf, size_t pack_bytes, hipStream_t stream)
{
    if (a.nF <= 0 || a.nS <= 0 || a.n_chunks <= 0 || a.t != 1 || a.d <= 0 || a.d > kMaxD || a.kind != KNM_KERNEL_GAUSSIAN)
        return hipErrorInvalidValue;
    if (a.chunk_len % kStage != 0 || a.n_chunks * a.chunk_len < a.nS || a.n_chunks > 65535) return hipErrorInvalidValue;
    switch (mfmas_of(a.d)) {
    case 2: return launch_nm<2>(a, pack_buf, pack_bytes, stream);
    case 3: return launch_nm<3>(a, pack_buf, pack_bytes, stream);
    case 4: return launch_nm<4>(a, pack_buf, pack_bytes, stream);
    case 5: return launch_nm<5>(a, pack_buf, pack_bytes, stream);
    default: return launch_nm<6>(a, pack_buf, pack_bytes, stream);
    }
}

} // namespace knm
