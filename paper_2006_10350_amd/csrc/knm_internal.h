// Internal declarations shared by the HIP sources of libknm (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <chrono>
#include <mutex>
#include <string>
#include <vector>

#include "knm.h"

namespace knm {

// ---- tile engine (knm_tile.hip) ---------------------------------------------------
//
// One engine serves both sweeps of K_nm^T (K_nm v) because the Gaussian kernel is
// symmetric in its two arguments:
//   out[f] = sum_s k(F_f, S_s) * vec[s]
// with "fixed" points F held in registers as the MFMA A operand and "stream" points S
// staged through LDS as the B operand.  Row sweep: F = X, S = C, vec = v.  Column
// sweep: F = C, S = X, vec = w, with the stream cut into chunks whose partial results
// are merged afterwards in a fixed order.
struct SweepArgs {
    const float *F;   // fixed points, nF x d, leading dimension ldf
    int64_t nF, ldf;
    const float *S;   // stream points, nS x d, leading dimension lds
    int64_t nS, lds;
    int d;
    // common shift of both point sets, d floats: the engines work with F - mu and S - mu (the kernels
    // depend on differences only), which keeps the norm terms of the expansion small for data that
    // is not centred; mu[d] != 0 says that the shift is not all zero
    const float *mu;
    const float *vec; // stream-side vectors: column c of stream point i is vec[i * ldv + c]
    int64_t ldv;
    int t;            // columns handled by this launch (1 for the register-resident engine)
    const float *wgt; // optional per-stream-point weight multiplied into vec (may be null)
    float *out;       // out[chunk * chunk_stride + f * ldo + c]
    // K-loop engines only: if not null the results go here instead, same indexing, in fp64 (the
    // register-resident engines ignore it and must be given `out`)
    double *out64 = nullptr;
    int64_t ldo, chunk_stride;
    int64_t chunk_len; // stream points per chunk (multiple of the stage size)
    int64_t n_chunks;
    // split-fp16 engines: incremented once per converted point whose scaled features or norm term lie
    // outside what the fp16 operands represent (|z| > 65000, |z|^2 / 2 >= 2^21, or not finite) and
    // were clamped; never null
    unsigned int *range_count;
    float sigma;      // length scale the engines work with (for the Laplacian kernel the caller's, rescaled)
    int kind;         // knm_kernel_kind (the kernels of r = |x - c|: K-loop engines only)
    // K-loop split-fp16 engine, reduction on the matrix cores: room of gemm_f16_vector_image_bytes() for the
    // vectors converted once per sweep into the layout of the LDS stage; null = every workgroup converts
    // the rows of its tiles itself
    void *vimg = nullptr;
    // split-fp16 engines: packed images of all stream (and, K-loop engine, all fixed) points kept by the caller for several
    // sweeps (SweepShare); an image that is not ready yet is packed by the sweep.  null: images live in the workspace
    // the launcher is given, slab by slab if need be
    void *fimg = nullptr, *simg = nullptr;
    bool fimg_ready = false, simg_ready = false;
    // K-loop engines: where the kernel values go, in blocks of 32 x 32, keep_s32 of them per 32 fixed points: in place of sums
    // (launch_keep_f16, and launch_sweep_gemm), or by rows beside the sums (launch_sweep_gemm_f16, Gaussian kernel, up to
    // kept_rows_max_t() columns on the vector ALU)
    float *keep = nullptr;
    int64_t keep_s32 = 0;
};

// ---- kept kernel values (knm_kept.hip) ------------------------------------------------
//
// Where forming the kernel values costs more than reading them from memory (d of a few hundred), the sweeps of a fit
// read them: all n x M of them in fp32, as the engine forms them, in blocks of 32 fixed x 32 stream
// points.  A block is 256 units of 16 bytes, unit (f, rq, h) = rows 8 rq + 4 h ... + 3 of the stream for fixed point f (a quad
// of an accumulator's registers), placed so that the engine's stores and the reads along either side of the matrix
// take whole 128-byte lines.
constexpr int kKeptBlock = 1024; // floats of a block
__host__ __device__ constexpr int kept_unit(int f, int h) { return (f >> 2) * 32 + h * 4 + (f & 3); } // + 8 rq
constexpr int64_t kept_rows(int64_t n) { return (n + 255) / 256 * 256; }                // fixed points, padded
constexpr int64_t kept_stream_blocks(int64_t n) { return (n + 127) / 128 * 4; }         // blocks of stream points, padded
constexpr size_t kept_bytes(int64_t nF, int64_t nS)
{
    return (size_t)(kept_rows(nF) / 32) * (size_t)kept_stream_blocks(nS) * kKeptBlock * sizeof(float);
}
struct KeptArgs {
    const float *values;
    int64_t nF, nS;          // points of the two sides
    bool over_stream;        // the sum runs over the stream points (result over the fixed ones), else the other way round
    const float *vec;        // vec[i * t + c] of the points summed over
    int t;                   // columns, at most kept_max_t()
    const float *wgt;        // per point summed over, or null
    double *part;            // part[chunk * n_out * t + i * t + c]
    int chunks;              // from kept_chunks()
};
int kept_max_t();
int kept_chunks(int64_t nF, int64_t nS, bool over_stream, int t); // partial results of a sum
hipError_t launch_kept_sum(const KeptArgs &a, hipStream_t stream);
// A product's, of a slab of rows of X (the fixed points) against the centres.  The sums over the rows [row0, row0 + rows) are those of the sweep over the columns to the last bit: fp32 sums of the 64 rows
// 8 i + 4 h ... + 3 of a tile of 128, added in fp64 over a chunk of `chunk_len` rows, one fp32 partial per chunk.
constexpr int kKeptTile = 128;
constexpr int kept_rows_max_t() { return 12; }
struct KeptRowsArgs {
    const float *values; // rows [row0, row0 + rows), against nS centres
    int64_t row0, rows;  // row0 a multiple of 256
    int64_t n, nS;       // rows of X in all, centres
    const float *vec;    // vec[i * t + c] of row row0 + i (times its weight)
    int t;
    // 2 x nS x t each: sums so far of the chunk that began in an earlier slab, and of the one that goes on in the next
    const double *state_in;
    double *state_out;
    float *part;         // part[chunk * nS * t + ...]
    int64_t chunk_len;   // a multiple of kKeptTile
};
hipError_t launch_kept_rows(const KeptRowsArgs &a, hipStream_t stream);
// Sums with up to kept_many_max_t() columns over kept values, from the vectors' packed image (launch_vector_image) of the points summed over,
// in fp32 over chunks of chunk_len of them (a multiple of 128)
struct KeptManyArgs {
    const float *values;
    int64_t nF, nS;
    bool over_stream;
    const void *vimg;
    const uint32_t *colmax;
    int t;
    int64_t chunk_len;
    float *part; // part[chunk * part_stride + i * ldo + c]
    int64_t part_stride, ldo;
};
int kept_many_max_t();
hipError_t launch_kept_many(const KeptManyArgs &a, hipStream_t stream);
// forms the values only: a.keep from the images a.fimg, a.simg of kept_rows() points each (packed here unless ready)
hipError_t launch_keep_f16(const SweepArgs &a, hipStream_t stream);

// What the sweeps of one pair of point sets have in common: the shift and the packed images, computed by the first sweep that
// needs them.  A product shares them between its two sweeps, a fit over all its iterations.
struct SweepShare {
    ::knm_ctx *ctx;
    const float *P[2]; // the sets (X and C)
    int64_t n[2], ld[2];
    int d;
    float sigma;
    int t;                       // columns of the sweeps
    // the smaller set, as a whole: the common shift is that of its rows, also where P[0] goes through X in slabs
    const float *shift_P;
    int64_t shift_n, shift_ld;
    // a fit's or sparse product's: images of both engines kept in blocks of the pool; else (a product) those of the K-loop engine, whose
    // two sweeps need both of them, in the context's image workspace
    bool pooled;
    int cross_term = -1, kind = -1; // what the images were packed for
    bool decided = false;        // whether images are kept has been decided
    void *img[2] = {nullptr, nullptr};
    int64_t rows[2] = {0, 0};    // points an image has room for
    int64_t ready[2] = {0, 0};   // points packed so far
    // kernel values of the pair kept for all its sweeps (knm_kept.hip), formed by a sweep over the columns (the fixed points are
    // the centres) or over the rows
    int uses = 0;                // sweeps over the pair that will be made (0: values are not kept)
    bool keep_decided = false;
    void *keep = nullptr;
    bool keep_columns = false;
    int64_t keep_n[2] = {0, 0};  // fixed and stream points they were formed for
    float *slab = nullptr;       // a product's: the row sweep leaves its values here (KeptRowsArgs)
    SweepShare(::knm_ctx *ctx, const float *X, int64_t n, int64_t ldx, const float *C, int64_t M, int64_t ldc, int d, float sigma, int t,
               bool pooled);
    ~SweepShare();
    SweepShare(const SweepShare &) = delete;
    SweepShare &operator=(const SweepShare &) = delete;
    int which(const float *Q, int64_t m, int64_t l) const
    {
        for (int k = 0; k < 2; ++k)
            if (P[k] == Q && n[k] == m && ld[k] == l) return k;
        return -1;
    }
    // Whether a sweep of set f against set s is one over the pair's kernel values, or its transpose.  A set against itself (k(C, C) in a
    // logistic fit) is, only where the two sets are one and the same: with the base pointer alone in common (every tenth row of X
    // as the centres, or X the first rows of C) the values are others.
    bool pair(int f, int s) const { return f != s || (P[0] == P[1] && n[0] == n[1] && ld[0] == ld[1]); }
};

// ---- kernels of r = |x - c| (Laplacian, Matern) on the K-loop engines ---------------------
//
// The engines' accumulators hold x = -s2 |f - s|^2 (s2 = log2(e) / (2 sigma^2) of the rescaled
// sigma), formed as norms minus cross term; the kernel value is 2^-sqrt(|x|).  The cancellation
// leaves an absolute error of about 1e-7 sqrt(d) N in x (N = s2 |f|^2, the norm in the same units),
// which the square root turns into error / (2 sqrt(|x|)): harmless for ordinary pairs, but 1e-4 to
// 1e-3 for coincident or nearly coincident ones, and every Nystrom centre coincides with a data
// row.  Pairs whose |x| lies below the threshold at which that error reaches about 1e-5 get their
// exponent again from fp32 differences of the two rows (exact for coincident rows, relative
// rounding error otherwise).  Such pairs are rare, so the branch is almost never taken.
__device__ __forceinline__ float near_pair_threshold(float norm_term, int d)
{
    // relative part: 1e-7 sqrt(d) N of rounding in the fp32 accumulation, at least the 2.4e-7 N that
    // the split-fp16 product leaves out; absolute part: the 2^-24 to which that engine's norm slots
    // are rounded
    const float N = fabsf(norm_term);
    return fmaxf(fmaxf(2.5e-5f * (float)d, 2.5e-4f) * N * N, 1.0e-5f);
}
__device__ __forceinline__ float exact_exponent(const float *__restrict__ f, const float *__restrict__ s, int d,
                                                float s2)
{
    float q = 0.0f;
    for (int k = 0; k < d; ++k) {
        const float diff = f[k] - s[k];
        q = fmaf(diff, diff, q);
    }
    return -s2 * q;
}
// kernel value from the exponent x = -(log2(e) u)^2 held by the accumulators
template <int KIND>
__device__ __forceinline__ float radial_from_exponent(float x)
{
    const float y = __builtin_amdgcn_sqrtf(fabsf(x)); // log2(e) u
    const float e = __builtin_amdgcn_exp2f(-y);
    if constexpr (KIND == KNM_KERNEL_LAPLACIAN) return e;
    const float u = y * 0.6931471805599453f;
    if constexpr (KIND == KNM_KERNEL_MATERN32) return fmaf(u, e, e);
    return e * fmaf(u, fmaf(u, 1.0f / 3.0f, 1.0f), 1.0f); // KNM_KERNEL_MATERN52
}

// register-resident engine (knm_tile.hip): d <= small_max_d(), one column per launch
int small_max_d();
int64_t stage_points();                 // stream points staged per LDS buffer
int64_t fixed_per_block(int d);         // fixed points one workgroup covers
hipError_t launch_sweep(const SweepArgs &a, hipStream_t stream);
// same shapes with the cross term as three f16 MFMA products (knm_tile_f16.hip): d <= f16_max_d()
int f16_max_d();
int f16_radial_max_d(); // the same for the kernels of r = |x - c|
int64_t f16_stage_points(int d, int kind); // stream points staged per LDS buffer by that engine
size_t f16_pack_bytes_per_point(int d);
// pack_buf: device workspace for the packed stream image, at least one chunk's worth
hipError_t launch_sweep_f16(const SweepArgs &a, void *pack_buf, size_t pack_bytes, hipStream_t stream);
int f16_workgroups_per_cu(int d, int kind);
// the fp32 cross term of the Gaussian kernel in three bf16 parts (knm_tile_b16.hip)
bool b16_pays(double entries, int d); // also whether it takes d
int b16_workgroups_per_cu(int d);
size_t b16_pack_bytes_per_point(int d);
hipError_t launch_sweep_b16(const SweepArgs &a, void *pack_buf, size_t pack_bytes, hipStream_t stream);
// K-loop engine (knm_gemm.hip): any d, up to gemm_max_t() columns per launch
int gemm_max_t();
bool gemm_leading_dimension_ok(int64_t ld); // leading dimensions the fp32 K-loop engine can index
int64_t gemm_stage_points();
int64_t gemm_fixed_per_block();
hipError_t launch_sweep_gemm(const SweepArgs &a, hipStream_t stream);
// the same shapes with the cross term as three f16 MFMA products (knm_gemm_f16.hip); both
// operands are packed into the workspace, whole or slab by slab
size_t gemm_f16_pack_bytes_per_point(int d);
size_t gemm_f16_head_bytes(); // bytes of the workspace in front of the images
int gemm_f16_max_t(int kind); // columns per launch at most
int gemm_f16_group_t(int d, int t_left, int kind, bool with_vector_image); // columns the next launch should take
// bytes of the packed vector image of a launch with t columns over nS_padded stream points (0: no such image)
size_t gemm_f16_vector_image_bytes(int d, int t, int64_t nS_padded);
// colmax (gemm_f16_head_bytes()) and, unless null, the packed image vimg of n vectors with t columns (times wgt), padded to n_padded
hipError_t launch_vector_image(const float *vec, int64_t ldv, const float *wgt, int64_t n, int64_t n_padded, int t, uint32_t *colmax, void *vimg,
                               hipStream_t stream);
size_t vector_image_bytes(int t, int64_t n_padded);
int gemm_f16_workgroups_per_cu(int d, int t, int kind); // of a launch with t columns and the packed vector image
bool gemm_f16_matrix_reduction(int d, int t);           // the reduction against t columns runs on the matrix cores
// sums over the stream points run through a chunk in fp32 (else those of a tile are added in fp64)
bool gemm_f16_fp32_sums(int d, int t, int kind);
bool gemm_fp32_sums(int t);
size_t gemm_f16_min_pack_bytes(int64_t nF, int64_t nS_padded, int64_t chunk_len, int d);
hipError_t launch_sweep_gemm_f16(const SweepArgs &a, void *pack_buf, size_t pack_bytes, hipStream_t stream);
// out[j * ldo] = sum over chunks of part[chunk * chunk_stride + j * ldp], summed in fp64 in a fixed
// order; the partials are fp32 or (part64) fp64, the result goes to `out` or, if not null, to `out64`
hipError_t launch_merge(const float *part, const double *part64, int64_t n_chunks, int64_t chunk_stride, int64_t ldp,
                        float *out, double *out64, int64_t ldo, int64_t count, hipStream_t stream);

// small predictions in one launch (knm_direct.hip): d <= 128, t <= 16; sigma as the engines take it.  With direct_chunks() > 1 the result
// is in partials of n x t each, to be merged
bool direct_takes(float sigma); // of the caller
bool direct_wide(const float *C, int64_t ldc, int d); // rows of C can be read 16 bytes at a time
bool direct_pays(int64_t n, int64_t M, int d, int t, bool wide, int cross_term);
int direct_chunks(int64_t n, int64_t M, int t);
hipError_t launch_direct(const float *X, int64_t n, int64_t ldx, const float *C, int64_t M, int64_t ldc, int d, float sigma, int kind,
                         const float *V, int t, float *out, double *part, unsigned int *range_count, float inv2s2, hipStream_t stream);

// fp64 rank-k update of the upper triangle of C on the matrix cores (knm_dsyrk.hip):
//   C[i, j] = alpha sum_{k < K} w[k] a(i, k) a(j, k) + beta C[i, j] + shift [i == j],  i <= j < n,
// a(i, k) = A[k + i lda] (form_nt = 0) or A[i + k lda] (form_nt = 1); w may be null; with tri the
// operand is upper triangular (a(i, k) taken as 0 for k < i whatever is stored there) and the zero part
// of the contraction is skipped; with trans_c entry (i, j) goes to C[j + i ldc] (the lower triangle)
hipError_t launch_rank_k_upper(int form_nt, int64_t n, int64_t K, double alpha, const double *A, int64_t lda,
                               const double *w, int tri, double beta, double shift, double *C, int64_t ldc,
                               hipStream_t stream, int trans_c = 0);

// general fp64 product on the same kernel: C (ni x nj) = alpha sum_{k < K} a(i, k) b(j, k) + beta C with
// a(i, k) = A[k + i lda] (a_nt = 0) or A[i + k lda] (a_nt = 1) and b(j, k) = B[k + j ldb] (b_nt = 0) or
// B[j + k ldb] (b_nt = 1, only with a_nt = 1).  part: 0 stores all of C, 1 its entries with i <= j, 2 those with
// i >= j.  C must not overlap A or B, except (in_place) that C may be B with a_nt = 0 and ni = K <= 128, or A with
// a_nt = 1, b_nt = 0 and nj = K <= 128
hipError_t launch_gemm_f64(int a_nt, int64_t ni, int64_t nj, int64_t K, double alpha, const double *A, int64_t lda,
                           const double *B, int64_t ldb, double beta, double *C, int64_t ldc, hipStream_t stream,
                           int b_nt = 0, int part = 0, bool in_place = false);

// A leaf of the factorisations (knm_leaf.h): the nb x nb block at A, nb <= 128, and its factor's inverse W
struct LeafArgs {
    double *A;
    int64_t lda;
    int nb;
    double *W;
    int64_t ldw, pivot0;
    unsigned long long *bad;
    int lower;
};
// The update of rows by the K rows above them, C(i, j) -= sum_k a(i, k) a(j, k) for ni x nj entries from the leaf's block on, in its storage (part 1, or 2
// with lower), but for that block itself, and the leaf beside it, in one launch
bool leaf_hides_update(int64_t rows, int64_t cols, int64_t K); // where that is faster than one after the other
hipError_t launch_leaf_beside_update(const LeafArgs &leaf, int64_t ni, int64_t nj, int64_t K, const double *P, hipStream_t stream);

// The symmetric update as integer products modulo small numbers (knm_residue.hip).  An operand's rows i < n (over k < K <= residue_max_k(); a(i, k) as in
// launch_rank_k_upper, times w[k] if given, rows of a triangular one starting at k + k0 = i) become planes of residues and
// one exponent per row; an update takes those of the operand's rows along the contiguous index u of C and across it, v.
// `wanted` (a device word): planes of an operand whose exponents are there already, made only where it is not 0.
bool residue_pays(int64_t n, int64_t K, bool triangular); // of an update of n x n entries
size_t residue_image_bytes(int64_t n, int64_t K);
int64_t residue_max_k();
hipError_t launch_residue_image(int form_nt, int64_t n, int64_t K, const double *A, int64_t lda, const double *w, int tri, int64_t k0, int *exps,
                                void *img, hipStream_t stream, const int *wanted = nullptr);
// room for the residues of the sums of an update over u x v entries, at most `cap` but for one strip of tiles
size_t residue_bytes(int64_t u, int64_t v, size_t cap);
struct ResidueUpdate {
    const void *img_u, *img_v;
    const int *differ;       // a device word: img_u stands for both sides where it is 0 (null: as given)
    const int *exp_u, *exp_v;
    int64_t n, K;            // of the images
    int64_t u0, u1, v0, v1;  // C[u + v ldc] for u0 <= u < u1, v0 <= v < v1 (the firsts multiples of 256), u <= v, or u >= v with lower
    int lower, tri;
    int64_t k0;
    double alpha, beta, shift;
    double *C;
    int64_t ldc;
    void *bytes;
    size_t bytes_size;
};
hipError_t launch_residue_update(const ResidueUpdate &p, hipStream_t stream);
// magnitude = sqrt |w|, with_sign = that with the sign of w, *negative = whether there is one
hipError_t launch_signed_root(const double *w, int64_t n, double *magnitude, double *with_sign, int *negative, hipStream_t stream);

// Merging of block inverses: S holds sb x sb column-major blocks (sb a multiple of 128) with the inverses of the
// 128 x 128 diagonal blocks of an upper factor R (entry (i, j), i <= j, at R[i + j ld], or R[j + i ld] with lower);
// on return the upper triangle of every block is the inverse of R's sb x sb diagonal block (the last one ends at
// M), and what is below its diagonal is overwritten
hipError_t launch_merge_inverses(const double *R, int64_t ld, int lower, int64_t M, double *S, int sb, hipStream_t stream);

// Sparse inputs (knm_sparse.hip): the two sweeps of one (X, C, sigma) for CSR X and C, prepared once
// (structure check, norms, centre lists per feature, accumulators) and then applied any number
// of times; and the fp64 kernel matrix of CSR centres for the preconditioner.
struct SparseProducts {
    struct Impl;
    Impl *impl;
    SparseProducts();
    ~SparseProducts();
    SparseProducts(const SparseProducts &) = delete;
    SparseProducts &operator=(const SparseProducts &) = delete;
    int prepare(struct ::knm_ctx *ctx, const int64_t *x_indptr, const int64_t *x_indices, const float *x_values, int64_t n,
                const int64_t *c_indptr, const int64_t *c_indices, const float *c_values, int64_t M, int64_t d,
                float sigma, int uses); // uses: sweeps (and columns of them) that will be made
    int v(const float *V, int t, float *W);                       // W (n x t) = K V
    int t_w(const float *W, const float *wgt, int t, float *U);   // U (M x t) = K^T (wgt .* W)
};
int sparse_kmm(struct ::knm_ctx *ctx, const int64_t *c_indptr, const int64_t *c_indices, const float *c_values, int64_t M,
               int64_t d, float sigma, double jitter, double *K, int64_t ldk);

} // namespace knm

struct knm_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    // workspace grown on demand and kept until knm_destroy
    float *w_buf = nullptr;
    size_t w_bytes = 0;
    float *part_buf = nullptr;
    size_t part_bytes = 0;
    float *mu_buf = nullptr;   // common shift of the two point sets of a sweep (d floats)
    size_t mu_bytes = 0;
    float *pack_buf = nullptr; // packed operand images of the split-fp16 engines
    size_t pack_bytes = 0;
    float *vimg_buf = nullptr; // packed vector image of the K-loop split-fp16 engine's matrix-core reduction
    size_t vimg_bytes = 0;
    size_t pack_limit = 0;     // cap on the image workspace chosen by the caller; 0 = engine defaults
    unsigned int *range_count = nullptr; // device word: operands the split-fp16 engines had to clamp (see SweepArgs)
    // this device's copy of the library's static scratch array (address looked up at knm_create), and
    // the state of a call that draws its workspace from it instead of allocating
    unsigned char *static_ws = nullptr;
    bool static_mode = false;
    size_t static_used = 0;
    int cross_term = KNM_CROSS_F16X3;
    int kernel_kind = KNM_KERNEL_GAUSSIAN;
    // sparse inputs: most frequent features treated densely, at most (0: none)
    int sparse_head_max = 128;
    // timing
    bool timing = false;
    hipEvent_t ev[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};
    bool ev_used[5] = {false, false, false, false, false};
    double fit_seconds[4] = {0.0, 0.0, 0.0, 0.0}; // last falkon_fit: preconditioner, rhs, iterations, tail
    std::string last_error;
    hipEvent_t fit_ev[2] = {nullptr, nullptr}; // begin and end of a fit's iterations (created lazily by knm_solver.hip)
    // device blocks of the temporaries of fits and sparse products, kept between calls (see pool_take)
    struct PoolBlock {
        void *p;
        size_t bytes;
        bool used;
    };
    std::vector<PoolBlock> pool;
    knm::SweepShare *share = nullptr; // of the product or fit whose sweeps are being enqueued
    const knm::SweepShare *mu_owner = nullptr; // mu_buf holds the shift of this pair of sets
    size_t pool_idle = 0; // bytes of the blocks not in use
    std::chrono::steady_clock::time_point room_asked{}; // when the card was last found to have room_left
    bool room_left = true;
    // a product's kept kernel values and sums over them (prod_kept), in a block of the pool that stays in use between calls, so that it is
    // where a captured product writes; spare while no product runs, unless one was captured
    void *slab = nullptr;
    size_t slab_bytes = 0;
    bool slab_captured = false;
    // blocks in use that can be done without: where their owners keep the pointers.  When something else finds no
    // room, those of [0] (kernel values, pair lists) and then of [1] (images) go back and the pointers become null
    std::vector<void **> spare[2];
    std::mutex pool_lock;
    // second stream for the look-ahead of the blocked factorisation (created lazily by knm_solver.hip)
    hipStream_t aux_stream = nullptr;
};

namespace knm {
// Named range for profilers (rocprofv3 --marker-trace): the phases of a product or fit.  The marker
// library (librocprofiler-sdk-roctx.so, or libroctx64.so) is looked up at run time the first time a
// range opens, and only if the environment variable KNM_MARKERS is set to a non-empty value other
// than 0: libknm itself links the HIP runtime only, and a range costs nothing otherwise.
struct TraceRange {
    explicit TraceRange(const char *name);
    ~TraceRange();
    TraceRange(const TraceRange &) = delete;
    TraceRange &operator=(const TraceRange &) = delete;
    bool open;
};
int ensure(knm_ctx *ctx, float **buf, size_t *cur, size_t need);
// Temporaries of calls that allocate (fits, sparse products): blocks of the context's own, taken from it and given back to
// it, because hipMalloc and hipFree cost 10 to 80 us each (2.4 ms of a 9.5 ms sparse product), and far more for large blocks.  Work on a context is
// ordered by its stream, so a block can be given back while kernels that use it are still queued.  Idle blocks of more than
// 16 GiB in all are freed (4 GiB where a sixteenth of the card is not free), and knm_destroy frees the rest.
// hipMalloc, with the idle blocks and then the spare ones (knm_ctx::spare) given up if there is no room
hipError_t device_alloc(knm_ctx *ctx, size_t bytes, void **out);
// (kOptional: without giving up spare blocks; kForSpeed: and only where the card has room to spare)
enum class PoolUse { kNeeded, kOptional, kForSpeed };
hipError_t pool_take(knm_ctx *ctx, size_t bytes, void **out, PoolUse use = PoolUse::kNeeded);
void pool_drop(knm_ctx *ctx, void *p); // back to the device
size_t pool_idle_bytes(knm_ctx *ctx);
void pool_trim(knm_ctx *ctx, size_t idle); // idle blocks beyond that many bytes, the newest first
void pool_give(knm_ctx *ctx, void *p);
bool spare_add(knm_ctx *ctx, int phase, void **p); // false: no host memory for it
void spare_remove(knm_ctx *ctx, int phase, void **p);
int fail(knm_ctx *ctx, int status, const char *what, hipError_t e = hipSuccess);
// The sweeps enqueued until it goes out of scope belong to the pair of point sets (see SweepShare).
struct ShareScope {
    knm_ctx *ctx;
    SweepShare *before;
    explicit ShareScope(SweepShare &s) : ctx(s.ctx), before(s.ctx->share) { ctx->share = &s; }
    ~ShareScope() { ctx->share = before; }
    ShareScope(const ShareScope &) = delete;
    ShareScope &operator=(const ShareScope &) = delete;
};
// true if (d, t) runs on the K-loop engine, false for the register-resident one
bool use_gemm_engine(int d, int t, int cross_term, int kind);
// number of stream chunks for a sweep over nS stream points against nF fixed points
int64_t choose_chunks(int64_t nF, int64_t nS, int d, int t, int cross_term, int kind, int64_t *chunk_len);
// the same with the engine given that takes a sweep of the fp32 mode: three-part numbers or fp32 MFMA
int64_t choose_chunks_for(int64_t nF, int64_t nS, int d, int t, int cross_term, int kind, bool parts, int64_t *chunk_len);
int do_knm_v(knm_ctx *ctx, const float *X, int64_t n, int d, int64_t ldx, const float *C, int64_t M,
             int64_t ldc, float sigma, const float *V, int t, float *W);
// U = K^T (wgt .* W) as fp32 rows (U) or, if U64 is not null, as fp64 rows (M x t, row-major) that
// never pass through fp32 after the merge of the chunk partials
int do_knm_t_w(knm_ctx *ctx, const float *X, int64_t n, int d, int64_t ldx, const float *C, int64_t M,
               int64_t ldc, float sigma, const float *Wv, const float *wgt, int t, float *U, double *U64 = nullptr);

// A temporary from the context's pool.
struct DevBuf {
    void *p = nullptr;
    knm_ctx *owner = nullptr;
    DevBuf() = default;
    DevBuf(const DevBuf &) = delete;
    DevBuf &operator=(const DevBuf &) = delete;
    ~DevBuf() { free(); }
    void free()
    {
        if (p) pool_give(owner, p);
        p = nullptr;
    }
    void drop() // back to the device
    {
        if (p) pool_drop(owner, p);
        p = nullptr;
    }
    int alloc(knm_ctx *ctx, size_t bytes)
    {
        owner = ctx;
        const hipError_t e = pool_take(ctx, bytes, &p);
        return e == hipSuccess ? KNM_OK : fail(ctx, KNM_ALLOC, "hipMalloc", e);
    }
    bool alloc_for_speed(knm_ctx *ctx, size_t bytes) // false where the card has no room to spare
    {
        owner = ctx;
        return pool_take(ctx, bytes, &p, PoolUse::kForSpeed) == hipSuccess;
    }
    template <class T> T *as() { return static_cast<T *>(p); }
};
} // namespace knm
