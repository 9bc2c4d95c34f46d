// fp64 symmetric rank-k updates on the matrix cores: the bulk of the preconditioner's flop.
//
// Both factorisations of the preconditioner (Alg. 1, the two Cholesky lines) spend M^3 / 3 flop
// each in the third step of the block Cholesky column update (Sec. 4, block Cholesky
// paragraph; appendix on the out-of-core algorithms): the trailing matrix loses the product
// of the just-solved block row with itself.  The triangular product between them (the same
// algorithm's T T^T line, with the diagonal weights of Alg. 2's WeightedPreconditioner) is the
// same contraction over a triangular operand.  One kernel serves both:
//
//   C[i, j] = alpha * sum_{k in [k0(j), K)} w[k] * a(i, k) * a(j, k) + beta * C[i, j] + shift * [i == j],   i <= j < n
//
//   form TN:  a(i, k) = A[k + i * lda]   (block row of the factor: contraction index contiguous)
//   form NT:  a(i, k) = A[i + k * lda]   (columns of the triangular factor: row index contiguous)
//
// The result goes to the upper triangle of C, or (trans_c) mirrored to C[j + i * ldc], i <= j: the lower
// triangle of the same array.  The two factors of the preconditioner share one array that way (the
// first in the upper triangle, the transpose of the second two rows below it), and a triangular operand
// is masked below its diagonal while it is staged, because what lies there belongs to the other factor.
//
// and, with the triangle test and the patch enumeration switched off, the general product
//   C[i, j] = alpha * sum_k a(i, k) * b(j, k) + beta * C[i, j]   over a rectangular C with its own
// column operand b (always TN), which carries the first two steps of the column update (products
// with the rows above and with inverted diagonal blocks) and the merging of block inverses.
//
// A workgroup of 4 wavefronts owns a 128 x 128 tile of C, each wavefront a 64 x 64 piece as
// 4 x 4 accumulators of v_mfma_f64_16x16x4_f64 (smaller tiles where there are few of them, see the launcher).  Operand tiles (16 deep) are staged through
// LDS, double buffered, with the global loads issued a stage and a half ahead.  Two
// workgroups share a CU (72 KB of LDS and 4 x ~225 registers each), so that one runs while the
// other sits at its per-stage barrier: 256 x 128 tiles with one 8-wavefront workgroup per CU
// were 4 % slower.
//
// On this chip the fp64 matrix instruction and the vector ALU do not overlap: every VALU
// cycle of either wavefront of a SIMD is taken from the matrix pipe (8 dependent fp64 adds per
// 16 products cost 7 % in a micro-benchmark).  The loop is therefore written to issue next
// to no VALU work: operands are fetched with buffer loads whose range check replaces the
// bounds tests (rows past the matrix read zeros or neighbouring rows, and only ever reach
// entries of C that are not stored), per-thread offsets are computed once, the per-stage
// advance is scalar arithmetic on the buffer descriptor, and every LDS address is a fixed
// per-thread base plus an immediate.
//
// Workgroups are numbered so that the 64 that run together on an XCD (and share its L2) cover
// a 1024 x 1024 patch of C and re-use each other's operand rows.
#include <type_traits>

#include "knm_internal.h"
#include "knm_leaf.h"

namespace knm {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

constexpr int kThreads = 256; // four wavefronts, each a quarter of the tile
constexpr int kXcds = 8;
// Tile of TI x TJ entries of C.  LDS image of an operand tile: element (k, i) at k * stride + i, for the k-contiguous form at
// k * stride + (i ^ (k % 16)).  The strides are 16 mod 32 doubles, so the four 16-lane groups of an
// operand read (four consecutive k) fall on alternating halves of the banks; the XOR spreads
// the 16 k of one column, which the k-contiguous form writes at once, over 16 bank pairs.
template <int TI, int TJ> struct Tile {
    // contraction depth of a stage: the small tiles have a quarter of the products per k, so they take twice the
    // depth to cover the latency of the loads and the barrier; 64 x 64 ones, taken where there are many, do that with four
    // workgroups per CU instead of two (1280 rows, k = 1280, 5000 columns: 348 -> 320 us; symmetric, 5000 rows, k = 640: 393 -> 364)
    static constexpr int kTK = TI * TJ >= 128 * 128 || (TI == 64 && TJ == 64) ? 16 : 32;
    static constexpr int kSA = TI == 16 ? 16 : TI + 16, kSB = TJ == 16 ? 16 : TJ + 16;
    static constexpr int kWI = TI == 16 ? 1 : TJ == 16 ? 4 : 2, kWJ = 4 / kWI; // wavefronts along i and j
    static constexpr int kStageDoubles = kTK * (kSA + kSB);
};

struct RankKArgs {
    const double *A; // operand of the rows of C
    int64_t lda;
    int64_t extent;  // elements from A to one past the last one of the operand
    const double *B; // operand of the columns of C (= A for the symmetric update)
    int64_t ldb;
    int64_t extent_b;
    const double *w; // weights along the contraction, or null
    double *C;
    int64_t ldc;
    int64_t n, nj, K; // C is n x nj (nj = n for the symmetric update)
    double alpha, beta, shift;
    int tri;           // operand is upper triangular (what is stored below its diagonal is ignored): tile column j0 starts at k = j0
    int trans_c;       // store entry (i, j) at C[j + i * ldc]
    int part;          // general product: store all entries (0), those with i <= j (1) or those with i >= j (2)
    int skip;          // and no tile inside the first skip x skip entries
    int patch_i, patch_j; // tiles of a patch (symmetric update: patch_j = patch_i)
    int64_t n_patch_i; // general product: patches along i
    int64_t n_patches; // patches in all (symmetric update: the upper-triangular ones)
    // one level of the merging of block inverses (see launch_merge_inverses): blockIdx.y is the pair
    int merge;         // 0: not such a launch, 1: first product, 2: second
    int merge_h, merge_pairs, sb, lower;
    int64_t M;
};

// Stage loader of one operand: a (kTK x R) tile, kPer elements per thread in kPer / VEC loads of
// VEC consecutive doubles, held in registers between the buffer loads and the LDS stores.
// VEC = 2 needs every load 16-byte aligned (even leading dimension, 16-byte aligned operand).
//   TN (FORM 0): thread -> k = VEC (tid % (16 / VEC)) .. + VEC (contiguous in memory), rows tid / (16 / VEC) + kPass r
//   NT (FORM 1): thread -> rows VEC (tid % (R / VEC)) .. + VEC (contiguous in memory), k = tid / (R / VEC) + kStepK r
template <int FORM, int R, int VEC, int kTK> struct Fetch {
    static constexpr int kPer = kTK * R / kThreads;
    static constexpr int kLoads = kPer / VEC;
    static constexpr int kPass = kThreads / (kTK / VEC);  // TN: row advance per load
    static constexpr int kStepK = kThreads / (R / VEC);   // NT: k advance per load
    double v[kPer];        // element e of load r at v[r * VEC + e]
    unsigned voff[kLoads]; // byte offsets of this thread's loads from the stage base
    const double *base;    // uniform: first element of the current stage of this tile
    int64_t left;          // uniform: elements from base to the end of the operand
    int64_t stage;         // uniform: elements per stage advance
    int row, k;            // tile-relative row and k of element 0

    __device__ __forceinline__ int row_of(int r, int e) const { return FORM == 0 ? row + kPass * r : row + e; }
    __device__ __forceinline__ int k_of(int r, int e) const { return FORM == 0 ? k + e : k + kStepK * r; }

    __device__ __forceinline__ void init(const double *P, int64_t ld, int64_t extent, int64_t row0, int64_t kbeg)
    {
        const int tid = threadIdx.x;
        int64_t first;
        if (FORM == 0) {
            k = VEC * (tid % (kTK / VEC));
            row = tid / (kTK / VEC);
            first = kbeg + row0 * ld;
            stage = kTK;
        } else {
            row = VEC * (tid % (R / VEC));
            k = tid / (R / VEC);
            first = row0 + kbeg * ld;
            stage = kTK * ld;
        }
#pragma unroll
        for (int r = 0; r < kLoads; ++r)
            voff[r] = (unsigned)((FORM == 0 ? (int64_t)k_of(r, 0) + (int64_t)row_of(r, 0) * ld
                                            : (int64_t)row_of(r, 0) + (int64_t)k_of(r, 0) * ld) * 8);
        base = P + first;
        left = extent - first;
    }
    // issue the loads of the next stage; reads past the operand's last element return zero
    __device__ __forceinline__ void load()
    {
        // left > 0 for every stage that is loaded; the descriptor's range is 32 bits
        const unsigned records = ((uint64_t)left >> 29) != 0 ? 0xffffffffu : (unsigned)left * 8u;
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(base), 0, (int)records, 0x00020000);
#pragma unroll
        for (int r = 0; r < kLoads; ++r) {
            if (VEC == 1) {
                v[r] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)voff[r], 0, 0));
            } else {
                const d2 x = __builtin_bit_cast(d2, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)voff[r], 0, 0));
                v[2 * r] = x[0];
                v[2 * r + 1] = x[1];
            }
        }
        base += stage;
        left -= stage;
    }
    // the k-contiguous form can run past K inside the operand: zero k >= k_left (last stage only)
    __device__ __forceinline__ void mask_tail(int k_left)
    {
        if (FORM == 0) {
#pragma unroll
            for (int r = 0; r < kLoads; ++r)
#pragma unroll
                for (int e = 0; e < VEC; ++e)
                    if (k_of(r, e) >= k_left) v[r * VEC + e] = 0.0;
        }
    }
    // upper-triangular operand: zero the elements below the diagonal, row > k + delta in tile-relative
    // terms (delta = global k of the stage's first element minus global row of the tile's first row)
    __device__ __forceinline__ void mask_lower(int delta)
    {
#pragma unroll
        for (int r = 0; r < kLoads; ++r)
#pragma unroll
            for (int e = 0; e < VEC; ++e)
                if (row_of(r, e) > k_of(r, e) + delta) v[r * VEC + e] = 0.0;
    }
    // weights of the stage's k, fetched together with the operand (buffer loads: zero past K)
    static constexpr int kW = FORM == 0 ? VEC : kLoads;
    double wv[kW];
    __device__ __forceinline__ void load_weights(const double *w_stage, int64_t w_left)
    {
        const unsigned records = ((uint64_t)w_left >> 29) != 0 ? 0xffffffffu : (unsigned)w_left * 8u;
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(w_stage), 0, (int)records, 0x00020000);
#pragma unroll
        for (int q = 0; q < kW; ++q) {
            const int kk = FORM == 0 ? k + q : k + kStepK * q;
            wv[q] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, kk * 8, 0, 0));
        }
    }
    __device__ __forceinline__ void scale()
    {
#pragma unroll
        for (int r = 0; r < kLoads; ++r)
#pragma unroll
            for (int e = 0; e < VEC; ++e) v[r * VEC + e] *= wv[FORM == 0 ? e : r];
    }
    __device__ __forceinline__ void store(double *lds, int stride) const
    {
#pragma unroll
        for (int r = 0; r < kLoads; ++r) {
            if (FORM == 1 && VEC == 2) {
                *reinterpret_cast<d2 *>(lds + k_of(r, 0) * stride + row_of(r, 0)) = d2{v[2 * r], v[2 * r + 1]};
            } else {
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    const int i = row_of(r, e), kk = k_of(r, e);
                    lds[kk * stride + (FORM == 0 ? (i ^ (kk & 15)) : i)] = v[r * VEC + e];
                }
            }
        }
    }
};

// FA, FB: forms of the row and column operands; SYM: symmetric update (B = A, upper triangle of C
// only, triangular patch enumeration); otherwise the general product C = alpha a b^T + beta C
// The tile of workgroup `group` of kThreads threads, in 2 Tile::kStageDoubles entries of LDS.
template <int FA, int FB, bool WEIGHTED, int VEC, bool SYM, int TI, int TJ>
__device__ __forceinline__ void rank_k_tile(RankKArgs a, int64_t group, double *lds)
{
    constexpr int kTK = Tile<TI, TJ>::kTK, kSA = Tile<TI, TJ>::kSA, kSB = Tile<TI, TJ>::kSB;
    constexpr int kStageDoubles = Tile<TI, TJ>::kStageDoubles;
    constexpr int kWI = Tile<TI, TJ>::kWI, kWJ = Tile<TI, TJ>::kWJ;
    constexpr int kMI = TI / 16 / kWI, kMJ = TJ / 16 / kWJ; // 16 x 16 accumulators of a wavefront
    if (!SYM && a.merge != 0) {
        // pair (off, off + h) of block k of the inverses: A, B, C and the sizes from the arrays' bases
        const int64_t k0 = (int64_t)(blockIdx.y / a.merge_pairs) * a.sb;
        const int64_t nbk = (a.M - k0 < a.sb) ? a.M - k0 : a.sb;
        const int64_t h = a.merge_h, off = 2 * h * (int64_t)(blockIdx.y % a.merge_pairs);
        if (off + h >= nbk) return;
        const int64_t h2 = (nbk - off - h < h) ? nbk - off - h : h; // order of the second block of the pair
        double *const S = a.C + (k0 / a.sb) * (int64_t)a.sb * a.sb;
        a.n = h;
        a.nj = h2;
        if (a.merge == 1) { // R12 W22, kept below the diagonal of the block
            a.A += a.lower ? (k0 + off + h) + (k0 + off) * a.lda : (k0 + off) + (k0 + off + h) * a.lda;
            a.B = S + (off + h) + (off + h) * a.sb;
            a.C = S + (off + h) + off * a.sb;
            a.K = h2;
            a.extent = FA == 0 ? (h - 1) * a.lda + h2 : (h2 - 1) * a.lda + h;
            a.extent_b = (h2 - 1) * a.sb + h2;
        } else { // -W11 times it
            a.A = S + off + off * a.sb;
            a.B = S + (off + h) + off * a.sb;
            a.C = S + off + (off + h) * a.sb;
            a.K = h;
            a.extent = (h - 1) * a.sb + h;
            a.extent_b = (h - 1) * a.sb + h2;
        }
    }
    // workgroup -> patch -> tile: consecutive workgroup ids go to consecutive XCDs, so the
    // workgroups of one patch are those with equal id % 8 and equal (id / 8) / patch_wgs
    const int64_t g = group;
    const int64_t slot = g / kXcds;
    const int patch_wgs = a.patch_i * a.patch_j;
    const int64_t q = (slot / patch_wgs) * kXcds + g % kXcds;
    if (q >= a.n_patches) return;
    const int wq = (int)(slot % patch_wgs);
    int64_t i0, j0;
    if (SYM) {
        // q = pj (pj + 1) / 2 + pi, pi <= pj
        int64_t pj = (int64_t)((sqrt(8.0 * (double)q + 1.0) - 1.0) * 0.5);
        while (pj * (pj + 1) / 2 > q) --pj;
        while ((pj + 1) * (pj + 2) / 2 <= q) ++pj;
        const int64_t pi = q - pj * (pj + 1) / 2;
        i0 = (pi * a.patch_i + wq % a.patch_i) * TI;
        j0 = (pj * a.patch_i + wq / a.patch_i) * TJ;
        if (i0 >= a.n || j0 >= a.n || i0 > j0 + (TJ - 1)) return; // outside C or strictly below its diagonal
    } else {
        const int64_t pi = q % a.n_patch_i, pj = q / a.n_patch_i;
        i0 = (pi * a.patch_i + wq % a.patch_i) * TI;
        j0 = (pj * a.patch_j + wq / a.patch_i) * TJ;
        if (i0 >= a.n || j0 >= a.nj) return;
        if ((a.part == 1 && i0 > j0 + (TJ - 1)) || (a.part == 2 && j0 > i0 + (TI - 1))) return; // nothing to store
        if (i0 + TI <= a.skip && j0 + TJ <= a.skip) return;
    }

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int wi = (wave % kWI) * (TI / kWI), wj = (wave / kWI) * (TJ / kWJ);
    // (triangular factors of the merges: W22 ends at its column's diagonal, W11 starts at its row's)
    if (!SYM && a.merge == 1 && a.K > j0 + TJ) a.K = j0 + TJ;
    const int64_t kbeg = (SYM && a.tri) ? j0 : (!SYM && a.merge == 2) ? i0 : 0; // a multiple of kTK
    const int64_t span = (a.K - kbeg + kTK - 1) / kTK;
    const int stages = span > 0x7fffffff ? 0x7fffffff : (int)span; // launch_rank_k_upper bounds K

    d4 acc[kMI][kMJ];
#pragma unroll
    for (int m = 0; m < kMI; ++m)
#pragma unroll
        for (int nn = 0; nn < kMJ; ++nn) acc[m][nn] = d4{0.0, 0.0, 0.0, 0.0};

    // C[4 r + l / 16][l % 16] of a 16 x 16 block is entry r of lane l of its accumulator.  The small tiles, whose products take
    // no longer than a miss, read their part of C before them
    constexpr bool kEarlyC = !SYM && TI * TJ <= 64 * 64;
    auto entry = [&](int m, int nn, int r, double *&dst) { // false: not stored
        const int64_t j = j0 + wj + nn * 16 + (lane & 15);
        const int64_t i = i0 + wi + m * 16 + (lane >> 4) + 4 * r;
        if (j >= a.nj || i >= a.n || (SYM && i > j)) return false;
        if (!SYM && ((a.part == 1 && i > j) || (a.part == 2 && i < j))) return false;
        dst = a.trans_c ? a.C + j + i * a.ldc : a.C + i + j * a.ldc;
        return true;
    };
    double old[kEarlyC ? kMI : 1][kEarlyC ? kMJ : 1][4];
    auto read_c = [&]() {
        if constexpr (kEarlyC) {
#pragma unroll
            for (int m = 0; m < kMI; ++m)
#pragma unroll
                for (int nn = 0; nn < kMJ; ++nn)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        double *dst = nullptr;
                        old[m][nn][r] = a.beta != 0.0 && entry(m, nn, r, dst) ? *dst : 0.0;
                    }
        }
    };

    if (stages <= 0) read_c();
    if (stages > 0) {
        Fetch<FA, TI, VEC, kTK> fa;
        Fetch<FB, TJ, VEC, kTK> fb;
        fa.init(a.A, a.lda, a.extent, i0, kbeg);
        fb.init(a.B, a.ldb, a.extent_b, j0, kbeg);
        // operand registers of k-step ks of the stage in `buf`: lane l takes k = 4 ks + l / 16
        const int qk = lane >> 4, l15 = lane & 15;
        auto read_ops = [&](const double *buf, int ks, double (&av)[kMI], double (&bv)[kMJ]) {
            const int krow = ks * 4 + qk;
            const double *pa = buf + krow * kSA + wi + (FA == 0 ? (l15 ^ (krow & 15)) : l15);
            const double *pb = buf + kTK * kSA + krow * kSB + wj + (FB == 0 ? (l15 ^ (krow & 15)) : l15);
#pragma unroll
            for (int m = 0; m < kMI; ++m) av[m] = pa[m * 16];
#pragma unroll
            for (int nn = 0; nn < kMJ; ++nn) bv[nn] = pb[nn * 16];
        };
        auto products = [&](const double (&av)[kMI], const double (&bv)[kMJ]) {
#pragma unroll
            for (int m = 0; m < kMI; ++m)
#pragma unroll
                for (int nn = 0; nn < kMJ; ++nn)
                    acc[m][nn] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[m], bv[nn], acc[m][nn], 0, 0, 0);
        };
        // registers -> LDS for stage s (whose loads were issued earlier)
        const int k_total = (int)(a.K - kbeg);
        auto commit = [&](int s, double *buf) {
            const int k_left = k_total - s * kTK;
            if (k_left < kTK) {
                fa.mask_tail(k_left);
                fb.mask_tail(k_left);
            }
            if (SYM && a.tri) {
                // stages that still overlap the diagonal band of a tile's rows (the first few of a tile)
                const int64_t kk0 = kbeg + (int64_t)s * kTK;
                if (kk0 < i0 + TI) fa.mask_lower((int)(kk0 - i0));
                if (kk0 < j0 + TJ) fb.mask_lower((int)(kk0 - j0));
            }
            if (WEIGHTED) fb.scale();
            fa.store(buf, kSA);
            fb.store(buf + kTK * kSA, kSB);
        };

        const double *w_stage = WEIGHTED ? a.w + kbeg : nullptr;
        int64_t w_left = a.K - kbeg;
        auto fetch = [&]() {
            fa.load();
            fb.load();
            if (WEIGHTED) {
                fb.load_weights(w_stage, w_left);
                w_stage += kTK;
                w_left -= kTK;
            }
        };
        double av[2][kMI], bv[2][kMJ];
        fetch();
        commit(0, lds);
        if (stages > 1) fetch();
        read_c();
        __syncthreads();
        read_ops(lds, 0, av[0], bv[0]);
        // Per stage: the operands of a k-step are read while the products of the one before
        // run; the next stage's tile goes to the other LDS buffer in mid-stage (its loads were
        // issued a stage earlier) and the loads of the stage after that follow; the one
        // barrier sits before the last k-step, after which the first operands of the next
        // stage are read under the last products.  Two stages per trip keep the buffer
        // offsets compile-time constants.
        // The products have no side effects the compiler must order against LDS traffic or
        // barriers, and left alone it sinks them below the barrier, which then waits for the
        // LDS stores with nothing to run; the scheduling fences keep each group where it is.
        auto stage_body = [&](int s, const double *cur, double *nxt) {
            constexpr int kSteps = kTK / 4;
#pragma unroll
            for (int ks = 0; ks < kSteps; ++ks) {
                const int now = ks & 1, next = now ^ 1;
                if (ks + 2 == kSteps && s + 1 < stages) {
                    commit(s + 1, nxt);
                    if (s + 2 < stages) fetch();
                }
                if (ks + 1 == kSteps) __syncthreads();
                if (ks + 1 < kSteps) read_ops(cur, ks + 1, av[next], bv[next]);
                else if (s + 1 < stages) read_ops(nxt, 0, av[next], bv[next]);
                __builtin_amdgcn_sched_barrier(0);
                products(av[now], bv[now]);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        for (int s = 0; s < stages; s += 2) {
            stage_body(s, lds, lds + kStageDoubles);
            if (s + 1 < stages) stage_body(s + 1, lds + kStageDoubles, lds);
        }
    }

#pragma unroll
    for (int m = 0; m < kMI; ++m)
#pragma unroll
        for (int nn = 0; nn < kMJ; ++nn)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                double *dst = nullptr;
                if (!entry(m, nn, r, dst)) continue;
                double v = a.alpha * acc[m][nn][r];
                if constexpr (kEarlyC) v += a.beta * old[m][nn][r];
                else if (a.beta != 0.0) v += a.beta * *dst;
                if (SYM && i0 + wi + m * 16 + (lane >> 4) + 4 * r == j0 + wj + nn * 16 + (lane & 15)) v += a.shift;
                *dst = v;
            }
}

template <int FA, int FB, bool WEIGHTED, int VEC, bool SYM, int TI = 128, int TJ = 128>
__global__ __launch_bounds__(kThreads) void rank_k_upper_kernel(RankKArgs a)
{
    __shared__ double lds[2 * Tile<TI, TJ>::kStageDoubles];
    rank_k_tile<FA, FB, WEIGHTED, VEC, SYM, TI, TJ>(a, blockIdx.x, lds);
}

// A leaf (the first workgroup) beside the update of the rows it belongs to, which does not wait for it: one after the other the leaf
// had the chip to itself for 25 us of every 128 rows.  Only half of a workgroup's wavefronts have a tile's work, the others end at once.  Fits at
// M = 5000 (logistic) 34.7 -> 33.8 ms, M = 10000 61.2 -> 60.3 and 32.4 -> 31.7, M = 20000 270 -> 264.7.
template <int F, int VEC, int T>
__global__ __launch_bounds__(kLeafThreads) void leaf_beside_update_kernel(LeafArgs leaf, RankKArgs a)
{
    static_assert(2 * Tile<T, T>::kStageDoubles <= kLeafDoubles && kThreads <= kLeafThreads && kLeaf % T == 0, "");
    __shared__ double lds[kLeafDoubles];
    if (blockIdx.x == 0) {
        leaf_block(leaf, lds);
        return;
    }
    if (threadIdx.x >= kThreads) return;
    rank_k_tile<F, F, false, VEC, false, T, T>(a, (int64_t)blockIdx.x - 1, lds);
}

// A thread's byte offsets inside a stage must fit the 32-bit buffer offset.
bool stage_offsets_fit(int form_nt, int64_t ld, int rows, int depth)
{
    const int64_t span = form_nt ? (int64_t)depth * ld + rows : (int64_t)rows * ld + depth;
    return span * 8 < 0xffffffffLL;
}

// Small tiles below this many 128 x 128 ones (two waves of the two workgroups a CU holds): the few wide tiles of a small
// product leave compute units idle and each is a chain of four times the matrix instructions (33 us for a product over
// k = 128 against 9 us).  From 256 to 2048 the fits take the same time; without small tiles M = 5000 takes 68 ms per
// logistic fit instead of 56, M = 20000 371 ms per fit instead of 355.
constexpr int64_t kSmallTilesBelow = 1024;

// Of those products, 32 x 32 tiles where 64 x 64 ones are few (t64: their number), and up to a few more where they are short: a
// wavefront's 4 products per k are a chain of 256 cycles, which 32 x 32 tiles cut to a quarter.  Microseconds with 64 x 64 and 32 x 32: 128 rows,
// k = 384: 1200 columns 22.3 and 10.6, 5000 23.1 and 18.0; 512 rows, k = 2048: 2500 columns (320 tiles) 142 and 112, 3500 (440) 143 and 157;
// 512 rows, k = 512: 2500 columns 44.5 and 34.3, 5000 (632) 62.9 and 62.6, 8700 (1088) 98.9 and 114.7.
bool smallest_tiles(int64_t t64, int64_t K) { return t64 <= 400 || (K <= 512 && t64 <= 640); }

// Triangular products of up to this many 64 x 64 tiles (n = 1400) take 32 x 32 ones: a tile that starts at k = 0 is one chain over the whole of k, which
// a quarter of the matrix instructions and twice the depth of a stage make half as long (n = 1000: 46 -> 23 us).  The trailing updates of the
// factorisations run behind other work and lose by it (0.2 % of a fit).
constexpr int64_t kSmallestUpTo = 256;

// In-place products (128 rows, k = 128) of up to this many columns take 16 at a time, longer ones 32: two workgroups per CU hold 8192, and
// with 16 a wavefront's chain of matrix instructions is half as long (preconditioner at M = 1000 0.99 -> 0.94 ms, M = 5000 6.87 -> 6.69 ms).
constexpr int64_t kNarrowUpTo = 8192;

// Updates of at least so many entries and up to this many 64 x 64 tiles run beside the leaf.  The diagonal block, updated on its
// own first, takes 5 us (k = 128) to 10 (k = 384): as long as the whole update of 128 rows and 1000 to 2000 columns (M = 1000: 0.5 % slower per fit with
// no lower limit), half of it at 5000 (10 to 18 us), a third at 9000.  Beside the leaf two workgroups share a CU, by its LDS, in place of three or four,
// which costs long updates more than the leaf's 25 us: fits at M = 20000 264.7 ms up to 1280 tiles, 266.4 up to 700, 267.8 up to 2600, 270 without.
constexpr int64_t kHiddenFrom = 128 * 2048, kHiddenUpTo = 1280;

// Patch of tiles that the workgroups of one XCD take together: 8 x 8, smaller where there would be fewer than four
// per XCD (all XCDs busy counts for more than shared rows of the operands)
void choose_patch(int64_t tiles_i, int64_t tiles_j, int *patch_i, int *patch_j)
{
    int pi = 8, pj = 8;
    auto patches = [&]() { return ((tiles_i + pi - 1) / pi) * ((tiles_j + pj - 1) / pj); };
    while (pi > 1 && pi >= 2 * tiles_i) pi /= 2;
    while (pj > 1 && pj >= 2 * tiles_j) pj /= 2;
    while (pi * pj > 1 && patches() < 4 * kXcds) {
        if (pi >= pj) pi /= 2;
        else pj /= 2;
    }
    *patch_i = pi;
    *patch_j = pj;
}

} // namespace

hipError_t launch_rank_k_upper(int form_nt, int64_t n, int64_t K, double alpha, const double *A, int64_t lda,
                               const double *w, int tri, double beta, double shift, double *C, int64_t ldc,
                               hipStream_t stream, int trans_c)
{
    if (n <= 0) return hipSuccess;
    RankKArgs a;
    a.A = a.B = A;
    a.lda = a.ldb = lda;
    a.w = w;
    a.C = C;
    a.ldc = ldc;
    a.n = a.nj = n;
    a.K = K;
    a.alpha = alpha;
    a.beta = beta;
    a.shift = shift;
    a.tri = tri;
    a.trans_c = trans_c;
    a.extent = a.extent_b = K <= 0 ? 0 : (form_nt ? (K - 1) * lda + n : (n - 1) * lda + K);
    a.merge = 0;
    a.part = a.skip = 0;
    const int64_t big = (n + 127) / 128;
    const int64_t half = (n + 63) / 64;
    const int T = big * (big + 1) / 2 >= kSmallTilesBelow ? 128 : tri && half * (half + 1) / 2 <= kSmallestUpTo ? 32 : 64;
    const int64_t tiles = (n + T - 1) / T;
    choose_patch((tiles + 1) / 2, tiles, &a.patch_i, &a.patch_j); // half of the square of tiles
    if (a.patch_j < a.patch_i) a.patch_i = a.patch_j;
    a.patch_j = a.patch_i;
    const int64_t n_patch = (tiles + a.patch_i - 1) / a.patch_i;
    a.n_patch_i = n_patch;
    a.n_patches = n_patch * (n_patch + 1) / 2;
    const int64_t groups = (a.n_patches + kXcds - 1) / kXcds;
    const int64_t wgs = groups * kXcds * a.patch_i * a.patch_j;
    if (wgs > 0x7fffffffLL) return hipErrorInvalidValue;
    if (!stage_offsets_fit(form_nt, lda, T, 32) || K >= (int64_t)0x7fffffff * 16) return hipErrorInvalidValue;
    const dim3 grid((unsigned)wgs), block(kThreads);
    // 16-byte loads when every one of them is aligned: tile origins are multiples of 64
    const bool vec2 = lda % 2 == 0 && reinterpret_cast<uintptr_t>(A) % 16 == 0;
    auto launch = [&](auto form, auto weighted, auto vec) {
        constexpr int F = decltype(form)::value, V = decltype(vec)::value;
        constexpr bool WT = decltype(weighted)::value;
        if (T == 32) hipLaunchKernelGGL((rank_k_upper_kernel<F, F, WT, V, true, 32, 32>), grid, block, 0, stream, a);
        else if (T == 64) hipLaunchKernelGGL((rank_k_upper_kernel<F, F, WT, V, true, 64, 64>), grid, block, 0, stream, a);
        else hipLaunchKernelGGL((rank_k_upper_kernel<F, F, WT, V, true>), grid, block, 0, stream, a);
    };
    auto with_vec = [&](auto form, auto weighted) {
        if (vec2) launch(form, weighted, std::integral_constant<int, 2>{});
        else launch(form, weighted, std::integral_constant<int, 1>{});
    };
    auto with_weights = [&](auto form) {
        if (w) with_vec(form, std::true_type{});
        else with_vec(form, std::false_type{});
    };
    if (form_nt) with_weights(std::integral_constant<int, 1>{});
    else with_weights(std::integral_constant<int, 0>{});
    return hipGetLastError();
}

hipError_t launch_gemm_f64(int a_nt, int64_t ni, int64_t nj, int64_t K, double alpha, const double *A, int64_t lda,
                           const double *B, int64_t ldb, double beta, double *C, int64_t ldc, hipStream_t stream, int b_nt,
                           int part, bool in_place)
{
    if (b_nt && !a_nt) return hipErrorInvalidValue; // not instantiated
    if (ni <= 0 || nj <= 0) return hipSuccess;
    RankKArgs a;
    a.A = A;
    a.lda = lda;
    a.B = B;
    a.ldb = ldb;
    a.w = nullptr;
    a.C = C;
    a.ldc = ldc;
    a.n = ni;
    a.nj = nj;
    a.K = K;
    a.alpha = alpha;
    a.beta = beta;
    a.shift = 0.0;
    a.tri = 0;
    a.trans_c = 0;
    a.part = part;
    a.skip = 0;
    a.merge = 0;
    a.extent = K <= 0 ? 0 : (a_nt ? (K - 1) * lda + ni : (ni - 1) * lda + K);
    a.extent_b = K <= 0 ? 0 : (b_nt ? (K - 1) * ldb + nj : (nj - 1) * ldb + K);
    const int64_t big = ((ni + 127) / 128) * ((nj + 127) / 128);
    int TI = 128, TJ = 128;
    if (big < kSmallTilesBelow) {
        // in place: a tile must hold all of the entries that are computed from the operand rows it overwrites
        if (!in_place) TI = TJ = smallest_tiles(((ni + 63) / 64) * ((nj + 63) / 64), K) ? 32 : 64;
        else (a_nt ? TI : TJ) = (a_nt ? ni : nj) <= kNarrowUpTo ? 16 : 32;
    }
    if (in_place && (a_nt ? nj > 128 : ni > 128)) return hipErrorInvalidValue;
    const int64_t tiles_i = (ni + TI - 1) / TI, tiles_j = (nj + TJ - 1) / TJ;
    choose_patch(tiles_i, tiles_j, &a.patch_i, &a.patch_j);
    a.n_patch_i = (tiles_i + a.patch_i - 1) / a.patch_i;
    a.n_patches = a.n_patch_i * ((tiles_j + a.patch_j - 1) / a.patch_j);
    const int64_t groups = (a.n_patches + kXcds - 1) / kXcds;
    const int64_t wgs = groups * kXcds * a.patch_i * a.patch_j;
    if (wgs > 0x7fffffffLL) return hipErrorInvalidValue;
    if (!stage_offsets_fit(a_nt, lda, TI, 32) || !stage_offsets_fit(b_nt, ldb, TJ, 32) || K >= (int64_t)0x7fffffff * 16)
        return hipErrorInvalidValue;
    const dim3 grid((unsigned)wgs), block(kThreads);
    const bool vec2 = lda % 2 == 0 && ldb % 2 == 0 && reinterpret_cast<uintptr_t>(A) % 16 == 0 &&
                      reinterpret_cast<uintptr_t>(B) % 16 == 0;
    auto launch = [&](auto fa, auto fb, auto vec) {
        constexpr int FA = decltype(fa)::value, FB = decltype(fb)::value, V = decltype(vec)::value;
        if (TI == 128 && TJ == 128) hipLaunchKernelGGL((rank_k_upper_kernel<FA, FB, false, V, false>), grid, block, 0, stream, a);
        else if (TI == 64) hipLaunchKernelGGL((rank_k_upper_kernel<FA, FB, false, V, false, 64, 64>), grid, block, 0, stream, a);
        else if (TI == 32 && TJ == 32) hipLaunchKernelGGL((rank_k_upper_kernel<FA, FB, false, V, false, 32, 32>), grid, block, 0, stream, a);
        else if constexpr (FA == 1 && FB == 0) {
            if (TI == 16) hipLaunchKernelGGL((rank_k_upper_kernel<FA, FB, false, V, false, 16, 128>), grid, block, 0, stream, a);
            else hipLaunchKernelGGL((rank_k_upper_kernel<FA, FB, false, V, false, 32, 128>), grid, block, 0, stream, a);
        } else if constexpr (FA == 0 && FB == 0) {
            if (TJ == 16) hipLaunchKernelGGL((rank_k_upper_kernel<FA, FB, false, V, false, 128, 16>), grid, block, 0, stream, a);
            else hipLaunchKernelGGL((rank_k_upper_kernel<FA, FB, false, V, false, 128, 32>), grid, block, 0, stream, a);
        }
    };
    auto with_forms = [&](auto vec) {
        constexpr std::integral_constant<int, 0> tn{};
        constexpr std::integral_constant<int, 1> nt{};
        if (b_nt) launch(nt, nt, vec);
        else if (a_nt) launch(nt, tn, vec);
        else launch(tn, tn, vec);
    };
    if (b_nt && in_place) return hipErrorInvalidValue; // not instantiated
    if (vec2) with_forms(std::integral_constant<int, 2>{});
    else with_forms(std::integral_constant<int, 1>{});
    return hipGetLastError();
}

bool leaf_hides_update(int64_t rows, int64_t cols, int64_t K)
{
    if (rows < kLeaf || cols <= kLeaf || K <= 0 || rows * cols < kHiddenFrom) return false;
    return ((rows + 63) / 64) * ((cols + 63) / 64) <= kHiddenUpTo;
}

hipError_t launch_leaf_beside_update(const LeafArgs &leaf, int64_t ni, int64_t nj, int64_t K, const double *P, hipStream_t stream)
{
    if (leaf.nb != kLeaf) return hipErrorInvalidValue;
    const int form = leaf.lower;
    const int64_t ld = leaf.lda;
    RankKArgs a = {};
    a.A = a.B = P;
    a.lda = a.ldb = a.ldc = ld;
    a.C = leaf.A;
    a.n = ni;
    a.nj = nj;
    a.K = K;
    a.alpha = -1.0;
    a.beta = 1.0;
    a.part = leaf.lower ? 2 : 1;
    a.skip = kLeaf;
    a.extent = form ? (K - 1) * ld + ni : (ni - 1) * ld + K;
    a.extent_b = form ? (K - 1) * ld + nj : (nj - 1) * ld + K;
    const int T = smallest_tiles(((ni + 63) / 64) * ((nj + 63) / 64), K) ? 32 : 64;
    const int64_t tiles_i = (ni + T - 1) / T, tiles_j = (nj + T - 1) / T;
    choose_patch(tiles_i, tiles_j, &a.patch_i, &a.patch_j);
    a.n_patch_i = (tiles_i + a.patch_i - 1) / a.patch_i;
    a.n_patches = a.n_patch_i * ((tiles_j + a.patch_j - 1) / a.patch_j);
    const int64_t wgs = (a.n_patches + kXcds - 1) / kXcds * kXcds * a.patch_i * a.patch_j + 1;
    if (wgs > 0x7fffffffLL || !stage_offsets_fit(form, ld, T, 32)) return hipErrorInvalidValue;
    const bool vec2 = ld % 2 == 0 && reinterpret_cast<uintptr_t>(P) % 16 == 0;
    auto launch = [&](auto f, auto v) {
        constexpr int F = decltype(f)::value, V = decltype(v)::value;
        if (T == 32) hipLaunchKernelGGL((leaf_beside_update_kernel<F, V, 32>), dim3((unsigned)wgs), dim3(kLeafThreads), 0, stream, leaf, a);
        else hipLaunchKernelGGL((leaf_beside_update_kernel<F, V, 64>), dim3((unsigned)wgs), dim3(kLeafThreads), 0, stream, leaf, a);
    };
    auto with_form = [&](auto v) {
        if (form) launch(std::integral_constant<int, 1>{}, v);
        else launch(std::integral_constant<int, 0>{}, v);
    };
    if (vec2) with_form(std::integral_constant<int, 2>{});
    else with_form(std::integral_constant<int, 1>{});
    return hipGetLastError();
}

hipError_t launch_merge_inverses(const double *R, int64_t ld, int lower, int64_t M, double *S, int sb, hipStream_t stream)
{
    RankKArgs a = {};
    a.ldc = sb;
    a.sb = sb;
    a.M = M;
    a.lower = lower;
    a.C = S;
    a.beta = 0.0;
    const unsigned blocks = (unsigned)((M + sb - 1) / sb);
    if (!stage_offsets_fit(lower ? 0 : 1, ld, 64, 32)) return hipErrorInvalidValue;
    const bool vec2 = ld % 2 == 0 && reinterpret_cast<uintptr_t>(R) % 16 == 0; // (S is allocated, sb a multiple of 128)
    for (int h = 128; h < sb; h *= 2) {
        a.merge_h = h;
        a.merge_pairs = (sb + 2 * h - 1) / (2 * h);
        const bool smallest = smallest_tiles((int64_t)(h / 64) * (h / 64) * blocks * a.merge_pairs, h);
        const int tiles = h / (smallest ? 32 : 64);
        a.patch_i = a.patch_j = 1;
        a.n_patch_i = tiles;
        a.n_patches = (int64_t)tiles * tiles;
        const dim3 grid((unsigned)((a.n_patches + kXcds - 1) / kXcds * kXcds), blocks * (unsigned)a.merge_pairs);
        a.merge = 1;
        a.alpha = 1.0;
        a.trans_c = 1;
        a.A = R;
        a.lda = ld;
        a.ldb = sb;
        auto launch = [&](auto fa, auto fb, auto vec) {
            constexpr int FA = decltype(fa)::value, FB = decltype(fb)::value, V = decltype(vec)::value;
            if (smallest) hipLaunchKernelGGL((rank_k_upper_kernel<FA, FB, false, V, false, 32, 32>), grid, dim3(kThreads), 0, stream, a);
            else hipLaunchKernelGGL((rank_k_upper_kernel<FA, FB, false, V, false, 64, 64>), grid, dim3(kThreads), 0, stream, a);
        };
        constexpr std::integral_constant<int, 0> tn{};
        constexpr std::integral_constant<int, 1> nt{}, one{};
        constexpr std::integral_constant<int, 2> two{};
        if (lower && vec2) launch(tn, tn, two);
        else if (lower) launch(tn, tn, one);
        else if (vec2) launch(nt, tn, two);
        else launch(nt, tn, one);
        a.merge = 2;
        a.alpha = -1.0;
        a.trans_c = 0;
        a.lda = sb;
        launch(nt, nt, two);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

} // namespace knm
