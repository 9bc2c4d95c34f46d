// fp64 symmetric updates of the preconditioner as integer products modulo 15 small numbers (residue number system, Chinese
// remainder theorem), on the int8 matrix cores:
//
//   C[i, j] = alpha * sum_k w[k] a(i, k) a(j, k) + beta * C[i, j] + shift * [i == j],   i <= j
//
// (the trailing updates of the blocked Cholesky factorisations and the triangular product T D T^T between them, as
// rank_k_upper_kernel forms them on the fp64 matrix cores).  The scheme is the one published for emulating fp64 products by int8 ones (Ozaki,
// Uchino, Imamura, "Ozaki Scheme II: a GEMM-oriented emulation of floating-point matrix multiplication using an integer modular
// technique", 2025), in its plainest form:
//   1. Row i of a (over k) is scaled by a power of two so that its norm is at most 2^58 and rounded to integers X(i, k).  By
//      Cauchy and Schwarz every sum over k of X(i, k) X(j, k) lies within +-2^116.
//   2. X is reduced modulo 15 pairwise coprime numbers up to 256, whose product P is 2^117.4: 15 planes of int8.
//   3. Per modulus a product of int8 matrices with exact int32 sums (at most 65536 terms of 2^14), reduced modulo the same number:
//      one byte per entry of C and modulus.
//   4. The 15 bytes give the sum itself, as the fraction sum_s r_s c_s / m_s of P modulo 1 (c_s the inverse of P / m_s modulo m_s), added in
//      fixed point to 2^-80 and rounded to the nearest int64 in units of 2^-64, then scaled back and added to C in fp64.
// Only step 1 rounds, and it rounds relative to a row's norm: an entry of a that is at least 2^-5 of it keeps all of its 53 bits, a smaller one
// is off by at most 2^-58 of the norm, whatever its own size.  An entry of the sum is so off by about 2e-18 |a_i| |a_j|, where running fp64 sums
// are off by their own last bits, sum by sum:
// block rows of 1024 of the factors of kernel matrices of 6144 centres (normal, skewed and image-like rows at their usual length scales, and length
// scales 0.25 to 0.4 times those), rms 2e-18 to 8e-17 of |a_i| |a_j| in place of 4.4e-17 to 1.1e-15, largest 2.0e-16 to 5.8e-16 in place of 3.1e-15 to 1.1e-14, all
// entries together (2-norm) 2e-17 to 2.3e-16 in place of 5.5e-16 to 1.5e-15; triangular products 2.3e-18 to 3.9e-18 in place of 4.7e-17 to 8.9e-17 rms.
// What Cholesky factors are good for, T^T T = K_MM to a small multiple of 2^-53 of its diagonal, is measured by the rows' norms.  Entries of
// the sum that are far below them, of rows that are large where the other is small, have fewer correct digits of their own than fp64 sums would give them.
//
// The fp64 matrix cores reach 64 TFLOP/s on large updates; int8 has 64 times their rate, of which 15 moduli, the power limit (operands that
// are random bytes: 2.7e15 operations a second from registers, 1.9e15 with their loads) and the passes over the bytes leave 79 to 100.
#include <type_traits>

#include "knm_internal.h"

namespace knm {
namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kModuli = 15;
constexpr int kModulus[kModuli] = {256, 253, 251, 247, 241, 239, 233, 229, 227, 223, 217, 211, 199, 197, 193};
// With 14 moduli and 54 bits the operands' rounding, 3e-17 |a_i| |a_j|, was above that of fp64 sums where these are small: later block rows, narrow
// kernels, skewed rows.
constexpr int kNormBits = 58;
constexpr int kDead = -(1 << 30); // exponent of a row that is not finite

constexpr unsigned __int128 product_of_moduli()
{
    unsigned __int128 p = 1;
    for (int m : kModulus) p *= (unsigned)m;
    return p;
}
constexpr unsigned __int128 kProduct = product_of_moduli();
static_assert(kProduct > ((unsigned __int128)1 << (2 * kNormBits + 1)) + ((unsigned __int128)1 << 90), "sums of either sign, with the rounding of X");
// fraction c_s / m_s of modulus s in four digits of 20 bits (the sum of 15 bytes times a digit, and half of 2^16, fits 32 bits)
constexpr uint32_t fraction_digit(int s, int digit)
{
    const unsigned m = (unsigned)kModulus[s];
    const unsigned rest = (unsigned)((kProduct / m) % m);
    unsigned c = 1;
    while (rest * c % m != 1) ++c;
    const unsigned __int128 f = ((unsigned __int128)c << 80) / m; // c < m
    return (uint32_t)(f >> (20 * (3 - digit))) & 0xfffffu;
}
struct Fractions {
    uint32_t digit[kModuli][4];
};
constexpr Fractions make_fractions()
{
    Fractions f{};
    for (int s = 0; s < kModuli; ++s)
        for (int q = 0; q < 4; ++q) f.digit[s][q] = fraction_digit(s, q);
    return f;
}
__constant__ const Fractions kFractions = make_fractions();
// P 2^-64 as the sum of two doubles
constexpr double kScaleHi = (double)kProduct * 0x1p-64;
constexpr double kScaleLo = (double)((__int128)kProduct - (__int128)(unsigned __int128)(double)kProduct) * 0x1p-64;

constexpr int kTileU = 256, kTileV = 128; // tile of C: along its contiguous index, and across it
constexpr int kStageK = 64;               // contraction depth of an LDS stage
constexpr int kRing = 3;
constexpr int kCells = (kTileU + kTileV) / 32 * (kStageK / 32); // of 1 KB: 32 rows x 32 k
constexpr int kThreads = 256, kWaves = kThreads / 64;
constexpr int kBlocks = kTileU / 32 * (kTileV / 32); // 32 x 32 blocks of a tile
constexpr int kPatchU = 4, kPatchV = 8;              // tiles that an XCD's workgroups take together
constexpr int kXcds = 8;
constexpr int64_t kTileBytes = (int64_t)kTileU * kTileV;

// Remainders by fp64 arithmetic: x - m rint(x / m) of a whole x up to 2^58.  Numbers below 2^51 are rounded by adding 1.5 2^52, which leaves
// them, as integers, in the low bits.  1 / m is not exact: a quotient may be off by more than a half, the remainder by as much of m
// beyond it, and where that can leave -128 .. 127 m is taken off or added once more.
constexpr double kRound = 6755399441055744.0;
constexpr bool beyond_int8(int m, int bits) // (1 / m is a multiple of 2^-60 for m <= 256)
{
    const __int128 miss = (__int128)(uint64_t)((1.0 / (double)m) * 0x1p60) * m - ((__int128)1 << 60);
    const double most = 0.5 * m + (double)(miss < 0 ? -miss : miss) * (bits < 60 ? 1.0 / (double)((uint64_t)1 << (60 - bits)) : 1.0);
    return most >= 128.0 && m != 256;
}
__device__ __forceinline__ uint32_t remainder_bits(double x, double m, double inv)
{
    const double q = fma(x, inv, kRound) - kRound;
    return (uint32_t)__builtin_bit_cast(uint64_t, fma(-m, q, x) + kRound); // the low byte counts
}
template <int M> __device__ __forceinline__ uint32_t remainder_of(double x) // of an operand
{
    const uint32_t bits = remainder_bits(x, (double)M, 1.0 / (double)M);
    if constexpr (!beyond_int8(M, kNormBits)) return bits;
    const int v = (int)bits;
    return (uint32_t)(v > 127 ? v - M : v < -127 ? v + M : v);
}
// low bytes of four words as one
__device__ __forceinline__ uint32_t low_bytes(uint32_t a, uint32_t b, uint32_t c, uint32_t d)
{
    const uint32_t ab = __builtin_amdgcn_perm(b, a, 0x0c0c0400u), cd = __builtin_amdgcn_perm(d, c, 0x0c0c0400u);
    return __builtin_amdgcn_perm(cd, ab, 0x05040100u);
}

int64_t padded_rows(int64_t n) { return (n + kTileU - 1) / kTileU * kTileU; }
int64_t padded_k(int64_t k) { return (k + kStageK - 1) / kStageK * kStageK; }

// element k of row i: A[k + i lda] (FORM 0) or A[i + k lda] (FORM 1); with tri, rows start at k + k0 = i
template <int FORM>
__device__ __forceinline__ double element(const double *__restrict__ A, int64_t lda, int64_t i, int64_t k, const double *__restrict__ w, int tri,
                                          int64_t k0)
{
    if (tri && k + k0 < i) return 0.0;
    const double x = A[FORM == 0 ? k + i * lda : i + k * lda];
    return w != nullptr ? x * w[k] : x;
}

// Power of two by which row i is scaled: its norm becomes at most 2^58 and (but for rows of extreme magnitude) more than 2^57.
// In two launches, sums of squares and maxima of slices of k, then what they come to: every sum has one order.
// FORM 0: a wavefront per row and slice; FORM 1: 64 rows by four wavefronts, which share a slice.
constexpr int kSlices = 16;
template <int FORM>
__global__ __launch_bounds__(256) void residue_norms_kernel(const double *__restrict__ A, int64_t lda, int64_t n, int64_t K,
                                                            const double *__restrict__ w, int tri, int64_t k0, double *__restrict__ part)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __shared__ double sh[2][4][64];
    const int64_t i = FORM == 0 ? (int64_t)blockIdx.x * 4 + wave : (int64_t)blockIdx.x * 64 + lane;
    const int64_t slice = (K + kSlices - 1) / kSlices;
    const int64_t begin = blockIdx.y * slice, end = begin + slice < K ? begin + slice : K;
    double sum = 0.0, most = 0.0;
    bool bad = false;
    if (i < n) {
        // (the slice's rows that start behind it have nothing in it)
        const int64_t step = FORM == 0 ? 64 : 4;
        if (!tri || end + k0 > i) {
#pragma unroll 8
            for (int64_t k = begin + (FORM == 0 ? lane : wave); k < end; k += step) {
                const double x = fabs(element<FORM>(A, lda, i, k, w, tri, k0));
                bad |= !(x <= 1.7976931348623157e308);
                most = fmax(most, x);
                sum = fma(x, x, sum);
            }
        }
    }
    if (bad) most = INFINITY;
    if (FORM == 0) {
        for (int m = 32; m > 0; m >>= 1) {
            sum += __shfl_xor(sum, m);
            most = fmax(most, __shfl_xor(most, m));
        }
        if (lane != 0) return;
    } else {
        sh[0][wave][lane] = sum;
        sh[1][wave][lane] = most;
        __syncthreads();
        if (wave != 0) return;
        for (int q = 1; q < 4; ++q) {
            sum += sh[0][q][lane];
            most = fmax(most, sh[1][q][lane]);
        }
    }
    if (i >= n) return;
    part[(2 * blockIdx.y) * n + i] = sum;
    part[(2 * blockIdx.y + 1) * n + i] = most;
}
__global__ __launch_bounds__(256) void residue_scale_kernel(const double *__restrict__ part, int64_t n, int64_t K, int *__restrict__ exps)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double sum = 0.0, most = 0.0;
#pragma unroll
    for (int q = 0; q < kSlices; ++q) {
        sum += part[2 * q * n + i];
        most = fmax(most, part[(2 * q + 1) * n + i]);
    }
    int e = 0;
    if (most == INFINITY) e = kDead;
    else if (most > 0.0) {
        int p;
        if (sum > 1e-280 && sum < 1e280) {
            (void)frexp(sum * (1.0 + 1e-9), &p); // sum < 2^p
            p = (p + 1) >> 1;                    // norm <= 2^p
        } else {
            (void)frexp(most, &p);
            int half = 0; // norm <= most sqrt(K) < 2^(p + half)
            while (((int64_t)1 << (2 * half)) < K) ++half;
            p += half;
        }
        e = kNormBits - p;
    }
    exps[i] = e;
}

template <int S> __device__ __forceinline__ void write_residues(const double (&x)[16], u32x4 *out, int64_t plane)
{
    if constexpr (S < kModuli) {
        constexpr int m = kModulus[S];
        u32x4 u;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            u[q] = low_bytes(remainder_of<m>(x[4 * q]), remainder_of<m>(x[4 * q + 1]), remainder_of<m>(x[4 * q + 2]), remainder_of<m>(x[4 * q + 3]));
        out[S * plane] = u;
        write_residues<S + 1>(x, out, plane);
    }
}

// Planes of residues: the unit of row i and k = 16 h .. 16 h + 15 of a chunk of 32 is 16 bytes, 64 units (32 rows x 2) a cell of 1 KB, the cells
// of 32 rows one behind the other along k.  A wavefront makes a cell of every plane.
template <int FORM>
__global__ __launch_bounds__(kThreads) void residue_convert_kernel(const double *__restrict__ A, int64_t lda, int64_t n, int64_t K,
                                                                  const double *__restrict__ w, int tri, int64_t k0,
                                                                  const int *__restrict__ exps, int64_t row_blocks, int64_t k_chunks,
                                                                  u32x4 *__restrict__ img, const int *__restrict__ wanted)
{
    if (wanted != nullptr && *wanted == 0) return;
    const int lane = threadIdx.x & 63;
    const int64_t cell = (int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6);
    if (cell >= row_blocks * k_chunks) return;
    // neighbouring wavefronts along the contiguous index
    const int64_t block = FORM == 0 ? cell / k_chunks : cell % row_blocks;
    const int64_t chunk = FORM == 0 ? cell % k_chunks : cell / row_blocks;
    // (a tile of C starts at the later of its first rows, rounded down to a stage)
    if (tri && chunk * 32 + 32 + k0 <= block * 32 / kTileU * kTileU - kStageK) return;
    const int64_t i = block * 32 + (lane & 31), kb = chunk * 32 + (lane >> 5) * 16;
    double x[16];
    int e = i < n ? exps[i] : kDead;
#pragma unroll
    for (int q = 0; q < 16; ++q) x[q] = i < n && kb + q < K ? element<FORM>(A, lda, i, kb + q, w, tri, k0) : 0.0;
#pragma unroll
    for (int q = 0; q < 16; ++q) x[q] = e == kDead ? 0.0 : rint(ldexp(x[q], e));
    u32x4 *out = img + (block * k_chunks + chunk) * 64 + lane;
    write_residues<0>(x, out, row_blocks * k_chunks * 64);
}

struct ResidueArgs {
    const char *img_u, *img_v; // planes of the two sides (along the contiguous index of C, and across)
    const int *differ;         // where it is 0 both sides are img_u (null: as given)
    int64_t plane;             // bytes of a plane
    int64_t k_chunks;          // of 32
    int64_t u0, v0;            // first row of a strip on either side, multiples of kTileU
    int64_t nu, nv;            // tiles of the strip
    int64_t patches_u, patches;
    int lower;                 // keep u >= v (else u <= v)
    int tri;                   // rows start at k + k0 = their index
    int64_t k0;
    uint8_t *bytes;            // [modulus][tile][block][lane][16]
    // combination
    const int *exp_u, *exp_v;
    int64_t n;
    double alpha, beta, shift;
    double *C;
    int64_t ldc;
};

__device__ __forceinline__ bool tile_kept(const ResidueArgs &a, int64_t u, int64_t v)
{
    return a.lower ? u + (kTileU - 1) >= v : u <= v + (kTileV - 1);
}

template <int S = 0> __device__ __forceinline__ void modulus_of(int s, double &m, double &inv)
{
    if constexpr (S < kModuli) {
        if (s == S) {
            m = (double)kModulus[S];
            inv = 1.0 / (double)kModulus[S];
        }
        modulus_of<S + 1>(s, m, inv);
    }
}

// One tile of C modulo one number per workgroup: 256 x 128, four wavefronts of 128 x 64, contraction in stages of 64 through a ring of three
// in LDS that loads which write LDS directly fill two stages ahead.  Two workgroups per CU.  Bound by the int8 matrix cores at the power
// limit: n = 17408, k = 2560 5.5 ms with 14 moduli, 4.0 with operands of zeros.  256 x 256 tiles, by eight wavefronts or by four of 128 x 128, which read a third
// less through the L2, took as long or 3 % longer.
__global__ __launch_bounds__(kThreads, 2) void residue_gemm_kernel(ResidueArgs a)
{
    __shared__ i32x4 ring[kRing][kCells][64];
    // workgroup -> modulus and patch -> tile: those of a patch run on one XCD together
    const int64_t g = blockIdx.x, slot = g / kXcds;
    constexpr int kPatch = kPatchU * kPatchV;
    const int64_t q = (slot / kPatch) * kXcds + g % kXcds;
    if (q >= a.patches * kModuli) return;
    const int s = (int)(q / a.patches);
    const int64_t patch = q % a.patches;
    const int w = (int)(slot % kPatch);
    const int64_t ut = (patch % a.patches_u) * kPatchU + w % kPatchU, vt = (patch / a.patches_u) * kPatchV + w / kPatchU;
    if (ut >= a.nu || vt >= a.nv) return;
    const int64_t u0 = a.u0 + ut * kTileU, v0 = a.v0 + vt * kTileV;
    if (!tile_kept(a, u0, v0)) return;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int64_t k_first = 0;
    if (a.tri) {
        k_first = (u0 > v0 ? u0 : v0) - a.k0;
        k_first = k_first > 0 ? k_first / kStageK : 0;
    }
    const int64_t total = a.k_chunks / 2;
    const int stages = (int)(total > k_first ? total - k_first : 0);

    // cells 0 .. 15: side u, (block of 32 rows, half of the stage); 16 .. 23: side v
    const int64_t row_bytes = a.k_chunks * 1024;
    const char *base_u = a.img_u + (int64_t)s * a.plane + (u0 / 32) * row_bytes + k_first * 2048;
    const char *const img_v = a.differ != nullptr && *a.differ == 0 ? a.img_u : a.img_v;
    const char *base_v = img_v + (int64_t)s * a.plane + (v0 / 32) * row_bytes + k_first * 2048;
    constexpr int kPerWave = kCells / kWaves;
    const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) i32x4 *)&ring[0][0][0]);
    unsigned offset[kPerWave]; // from the side's base
#pragma unroll
    for (int c = 0; c < kPerWave; ++c) {
        const int cell = wave * kPerWave + c, own = cell < 16 ? cell : cell - 16;
        offset[c] = (unsigned)((own >> 1) * row_bytes + (own & 1) * 1024) + (unsigned)lane * 16u;
    }
    auto issue = [&](int c, int stage, int slot_of) { // cell c of this wavefront's
        const int cell = wave * kPerWave + c;
        const uint64_t p = (uint64_t)((cell < 16 ? base_u : base_v) + (int64_t)stage * 2048);
        const unsigned l = __builtin_amdgcn_readfirstlane(lds0 + (unsigned)(slot_of * kCells + cell) * 1024u);
        const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)p), hi = __builtin_amdgcn_readfirstlane((unsigned)(p >> 32));
        unsigned keep;
        // (one wait state between a scalar write of M0 and the load that reads it)
        asm volatile("s_mov_b32 %[keep], m0\n\ts_mov_b32 m0, %[l]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[o], %[b]\n\ts_mov_b32 m0, %[keep]"
                     : [keep] "=&s"(keep)
                     : [l] "s"(l), [o] "v"(offset[c]), [b] "s"(((uint64_t)hi << 32) | lo)
                     : "memory");
    };

    i32x16 acc[4][2]; // blocks of 32 along u, along v
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[x][y][r] = 0;
    const int wu = (wave & 1) * 4, wv = (wave >> 1) * 2; // first blocks of the wavefront

    i32x4 side_u[2][4], side_v[2][2];
    auto read = [&](int q, int slot_of, int h) { // operand q of 6
        if (q < 2) side_v[h][q] = ring[slot_of][16 + (wv + q) * 2 + h][lane];
        else side_u[h][q - 2] = ring[slot_of][(wu + q - 2) * 2 + h][lane];
    };
    // the products of half a stage, with other work issued between them
    auto multiply = [&](int h, auto between) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            acc[k >> 1][k & 1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(side_v[h][k & 1], side_u[h][k >> 1], acc[k >> 1][k & 1], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            between(k);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    for (int st = 0; st < 2 && st < stages; ++st)
#pragma unroll
        for (int c = 0; c < kPerWave; ++c) issue(c, st, st);
    int cur = 0;
    for (int st = 0; st < stages; ++st) {
        // stage st has landed when no more loads are under way than the next one's
        if (st + 1 < stages) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kPerWave) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads(); // everyone's share has, and the slot of the stage before this one is free
        const int before = cur == 0 ? kRing - 1 : cur - 1;
#pragma unroll
        for (int q = 0; q < 6; ++q) read(q, cur, 0);
        __builtin_amdgcn_sched_barrier(0);
        multiply(0, [&](int k) {
            if (k < 6) read(k, cur, 1);
        });
        const bool load = st + 2 < stages;
        multiply(1, [&](int k) {
            if (k < 6 && load) issue(k, st + 2, before);
        });
        cur = cur == kRing - 1 ? 0 : cur + 1;
    }

    double m = 256.0, inv = 1.0 / 256.0;
    modulus_of(s, m, inv);
    u32x4 *out = reinterpret_cast<u32x4 *>(a.bytes) + (((int64_t)s * a.nu * a.nv + vt * a.nu + ut) * kBlocks) * 64 + lane;
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            u32x4 packed;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const auto &v = acc[x][y];
                packed[r] = low_bytes(remainder_bits((double)v[4 * r], m, inv), remainder_bits((double)v[4 * r + 1], m, inv),
                                      remainder_bits((double)v[4 * r + 2], m, inv), remainder_bits((double)v[4 * r + 3], m, inv));
            }
            out[((wu + x) * (kTileV / 32) + wv + y) * 64] = packed;
        }
}

// The sums from their residues, and C from them: a wavefront per 32 x 32 block.  Bound by memory: 15 bytes read, C read and written.
__global__ __launch_bounds__(kThreads) void residue_combine_kernel(ResidueArgs a)
{
    const int lane = threadIdx.x & 63;
    const int64_t id = (int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6);
    const int64_t tile = id / kBlocks;
    const int block = (int)(id % kBlocks);
    if (tile >= a.nu * a.nv) return;
    const int64_t tu = a.u0 + (tile % a.nu) * kTileU, tv = a.v0 + (tile / a.nu) * kTileV;
    const int64_t bu = tu + (block / (kTileV / 32)) * 32, bv = tv + (block % (kTileV / 32)) * 32;
    if (!tile_kept(a, tu, tv) || bu >= a.n || bv >= a.n || (a.lower ? bu + 31 < bv : bu > bv + 31)) return;
    const u32x4 *in = reinterpret_cast<const u32x4 *>(a.bytes) + (tile * kBlocks + block) * 64 + lane;
    const int64_t plane = a.nu * a.nv * kBlocks * 64;
    u32x4 r[kModuli];
#pragma unroll
    for (int s = 0; s < kModuli; ++s) r[s] = in[s * plane];
    const int64_t u = bu + (lane & 31);
    const int eu = u < a.n ? a.exp_u[u] : 0;
    // (register e of a lane: row 8 (e / 4) + 4 (lane / 32) + e % 4 of side v)
    double old[16];
    int ev[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int64_t v = bv + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
        const bool in_c = u < a.n && v < a.n && (a.lower ? u >= v : u <= v);
        old[e] = in_c && a.beta != 0.0 ? a.C[u + v * a.ldc] : 0.0;
        ev[e] = v < a.n ? a.exp_v[v] : 0;
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        int d[4] = {0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < kModuli; ++s) {
            const int b = (int8_t)(r[s][e >> 2] >> (8 * (e & 3)));
#pragma unroll
            for (int k = 0; k < 4; ++k) d[k] += __mul24(b, (int)kFractions.digit[s][k]);
        }
        // the digits' sums as a fraction of 2^64, modulo 1
        const uint64_t f = ((uint64_t)(int64_t)d[0] << 44) + ((uint64_t)(int64_t)d[1] << 24) + ((uint64_t)(int64_t)d[2] << 4) + (uint64_t)(int64_t)((d[3] + 32768) >> 16);
        const double c = (double)(int64_t)f;
        double sum = fma(c, kScaleLo, c * kScaleHi);
        sum = eu == kDead || ev[e] == kDead ? __builtin_nan("") : ldexp(sum, -(eu + ev[e]));
        const int64_t v = bv + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
        if (u >= a.n || v >= a.n || (a.lower ? u < v : u > v)) continue;
        double x = a.alpha * sum;
        if (a.beta != 0.0) x += a.beta * old[e];
        if (u == v) x += a.shift;
        a.C[u + v * a.ldc] = x;
    }
}

__global__ void clear_word_kernel(int *word) { *word = 0; }
// (negative: raised where a weight has a sign; it may not be a number either)
__global__ void signed_root_kernel(const double *__restrict__ w, int64_t n, double *__restrict__ magnitude, double *__restrict__ with_sign,
                                   int *__restrict__ negative)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const double x = w[k], r = sqrt(fabs(x));
    magnitude[k] = r;
    with_sign[k] = x < 0.0 ? -r : r;
    if (x < 0.0) atomicOr(negative, 1);
}

} // namespace

// Microseconds measured: 127e6 flop each for the int8 products, 49 bytes an entry of C at 6 TB/s, 23 an element of the operand at 3.2, launches;
// the fp64 matrix cores 50e6 to 64e6 flop.  n = 17408, k = 2560: 12.2 -> 7.7 ms; 8704, 1280: 2.0 -> 1.2; 4352, 1024: 0.44 -> 0.30.  Triangular products
// go by it from 3488 centres on, block rows from 5304.
bool residue_pays(int64_t n, int64_t K, bool triangular)
{
    if (K <= 0 || n <= 0) return false;
    const double entries = 0.5 * (double)n * (double)n, elements = (double)n * (double)K * (triangular ? 0.5 : 1.0);
    const double flop = 2.0 * entries * (double)K * (triangular ? 1.0 / 3.0 : 1.0);
    return flop / 127e6 + entries * 49.0 / 6.0e6 + elements * 23.0 / 3.2e6 + 40.0 < 0.9 * flop / 52e6;
}

size_t residue_image_bytes(int64_t n, int64_t K) { return (size_t)kModuli * (size_t)padded_rows(n) * (size_t)padded_k(K); }
int64_t residue_max_k() { return 65536; } // sums of up to 2^30

hipError_t launch_residue_image(int form_nt, int64_t n, int64_t K, const double *A, int64_t lda, const double *w, int tri, int64_t k0, int *exps,
                                void *img, hipStream_t stream, const int *wanted)
{
    if (n <= 0 || K <= 0 || K > residue_max_k()) return hipErrorInvalidValue;
    const int64_t blocks = padded_rows(n) / 32, chunks = padded_k(K) / 32;
    const int64_t wgs = (blocks * chunks + kWaves - 1) / kWaves;
    if (wgs > 0x7fffffffLL) return hipErrorInvalidValue;
    double *part = static_cast<double *>(img); // (2 x 16 numbers a row, before the planes are written there)
    static_assert(2 * kSlices * sizeof(double) <= (size_t)kModuli * kStageK, "room for them");
    auto launch = [&](auto form) {
        constexpr int F = decltype(form)::value;
        if (wanted == nullptr) {
            hipLaunchKernelGGL((residue_norms_kernel<F>), dim3((unsigned)((n + (F ? 63 : 3)) / (F ? 64 : 4)), kSlices), dim3(256), 0, stream, A, lda, n,
                               K, w, tri, k0, part);
            hipLaunchKernelGGL(residue_scale_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, part, n, K, exps);
        }
        hipLaunchKernelGGL((residue_convert_kernel<F>), dim3((unsigned)wgs), dim3(kThreads), 0, stream, A, lda, n, K, w, tri, k0, exps, blocks,
                           chunks, static_cast<u32x4 *>(img), wanted);
    };
    if (form_nt) launch(std::integral_constant<int, 1>{});
    else launch(std::integral_constant<int, 0>{});
    return hipGetLastError();
}

// bytes of the residues of the widest strip of a region that fits `cap` (at least one column of tiles)
static int64_t strip_tiles(int64_t nu, int64_t nv, size_t cap)
{
    int64_t w = (int64_t)(cap / (size_t)(kTileBytes * kModuli * nu));
    w = w < 2 ? 2 : w / 2 * 2; // (whole tiles of the other side)
    const int64_t strips = (nv + w - 1) / w;
    return ((nv + strips - 1) / strips + 1) / 2 * 2; // of the same width
}
size_t residue_bytes(int64_t u, int64_t v, size_t cap)
{
    const int64_t nu = (u + kTileU - 1) / kTileU, nv = (v + kTileV - 1) / kTileV;
    return (size_t)(kTileBytes * kModuli) * (size_t)(nu * strip_tiles(nu, nv, cap));
}

hipError_t launch_residue_update(const ResidueUpdate &p, hipStream_t stream)
{
    if (p.u0 % kTileU != 0 || p.v0 % kTileU != 0 || p.K <= 0 || p.K > residue_max_k()) return hipErrorInvalidValue;
    if (p.u1 <= p.u0 || p.v1 <= p.v0) return hipSuccess;
    ResidueArgs a;
    a.img_u = static_cast<const char *>(p.img_u);
    a.img_v = static_cast<const char *>(p.img_v);
    a.differ = p.differ;
    a.plane = padded_rows(p.n) * padded_k(p.K);
    a.k_chunks = padded_k(p.K) / 32;
    a.lower = p.lower;
    a.tri = p.tri;
    a.k0 = p.k0;
    a.bytes = static_cast<uint8_t *>(p.bytes);
    a.exp_u = p.exp_u;
    a.exp_v = p.exp_v;
    a.n = p.n;
    a.alpha = p.alpha;
    a.beta = p.beta;
    a.shift = p.shift;
    a.C = p.C;
    a.ldc = p.ldc;
    const int64_t all_u = (p.u1 - p.u0 + kTileU - 1) / kTileU, all_v = (p.v1 - p.v0 + kTileV - 1) / kTileV;
    const int64_t width = strip_tiles(all_u, all_v, p.bytes_size);
    if ((size_t)(kTileBytes * kModuli) * (size_t)(all_u * width) > p.bytes_size) return hipErrorInvalidValue;
    for (int64_t t = 0; t < all_v; t += width) {
        a.v0 = p.v0 + t * kTileV;
        a.nv = all_v - t < width ? all_v - t : width;
        a.u0 = p.u0;
        a.nu = all_u;
        // the part of the strip on the kept side of the diagonal
        if (p.lower) {
            if (a.v0 > a.u0) {
                const int64_t skip = (a.v0 - a.u0) / kTileU;
                a.u0 += skip * kTileU;
                a.nu -= skip;
            }
        } else {
            const int64_t last = (a.v0 + a.nv * kTileV - 1 - a.u0) / kTileU + 1; // tiles with a row u <= the strip's last v
            if (last < a.nu) a.nu = last;
        }
        if (a.nu <= 0) continue;
        a.patches_u = (a.nu + kPatchU - 1) / kPatchU;
        a.patches = a.patches_u * ((a.nv + kPatchV - 1) / kPatchV);
        const int64_t wgs = (a.patches * kModuli + kXcds - 1) / kXcds * kXcds * kPatchU * kPatchV;
        const int64_t cwgs = a.nu * a.nv * kBlocks / kWaves;
        if (wgs > 0x7fffffffLL || cwgs > 0x7fffffffLL) return hipErrorInvalidValue;
        hipLaunchKernelGGL(residue_gemm_kernel, dim3((unsigned)wgs), dim3(kThreads), 0, stream, a);
        hipLaunchKernelGGL(residue_combine_kernel, dim3((unsigned)cwgs), dim3(kThreads), 0, stream, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_signed_root(const double *w, int64_t n, double *magnitude, double *with_sign, int *negative, hipStream_t stream)
{
    // (cleared by a kernel: precond_residue_update may be captured into a graph, where memset nodes are to be avoided)
    hipLaunchKernelGGL(clear_word_kernel, dim3(1), dim3(1), 0, stream, negative);
    hipLaunchKernelGGL(signed_root_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, w, n, magnitude, with_sign, negative);
    return hipGetLastError();
}

} // namespace knm
