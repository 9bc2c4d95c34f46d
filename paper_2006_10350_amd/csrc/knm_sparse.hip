// Kernel product for sparse inputs (Sec. 4, "Dealing with sparse datasets"): X and C in CSR
// form with a feature dimension far beyond what a dense row can hold.
//
// The kernel matrix of sparse points is still dense, but most of it is a rank-one matrix:
// with a_i = exp(-|x_i|^2 / 2 sigma^2), b_j = exp(-|c_j|^2 / 2 sigma^2) and g_ij = x_i . c_j,
//   K_ij = a_i b_j exp(g_ij / sigma^2),
// and g_ij = 0 unless the two points share a feature.  So
//   (K v)_i   = a_i sum_j b_j v_j  +  sum_{j : g_ij != 0} (K_ij - a_i b_j) v_j
//   (K^T w)_j = b_j sum_i a_i w_i  +  sum_{i : g_ij != 0} (K_ij - a_i b_j) w_i,
// exactly (up to rounding order), and only the pairs that share a feature are ever visited:
// no dense n x M sweep, no dense tile of the cross term.  The paper forms the dense kernel
// blocks from a sparse matrix product; this is the same result with the all-ones part of
// exp(g / sigma^2) summed in closed form.
//
// One wavefront owns a row of X at a time and a private dense accumulator over the M centres
// (in HBM / L2): it walks the row's features, and for each feature the list of centres that
// have it (C transposed to CSC once per call), adding x_if c_jf into the accumulator; a second
// walk takes every touched entry out again (atomic exchange with zero, so a centre reached
// through several features is consumed once), turns it into K_ij - a_i b_j and adds it to the
// row's sum (row sweep) or scatters it into a fp64 image of U (column sweep, fp64 atomics: the
// summation order varies from run to run, which the rounding to fp32 at the end mostly hides).  Its lists are walked end to end,
// 64 updates at a time.  The additions are the hardware's
// fp32 atomic add (the accumulators and U live in ordinary device memory).
//
// What a row has to walk is prepared once per (X, C): a work list with the start and length of
// the centre list of every entry whose feature occurs in a centre at all.  A row with few pair
// updates accumulates in a small table in LDS instead of the accumulator in device memory.  Where
// both directions or several sweeps are wanted, one walk writes the pairs down and the sweeps
// read them (kMaxPairs below).  The few features that
// occur in a large share of the centres are not walked: their pairs are covered by one dense
// product over those features (see "head features" below), which takes the place of the
// rank-one term.
#include <algorithm>
#include <cstring>
#include <memory>
#include <new>
#include <vector>

#include "knm_internal.h"

namespace knm {
namespace {

constexpr int kSpThreads = 256;
constexpr int kSpWaves = kSpThreads / 64;
constexpr int kScanChunk = 4096;  // elements per workgroup of the prefix sum
// Rows of C per launch that takes the places in the lists: no more than 64 entries of an average list span, which update neighbouring
// accumulators then, between 512 and 4096.  20000 centres of 100 entries: 0.27 ms with 1024 rows, 0.17 with 4096; the walks take the same time up to d
// = 4e5, and within the 2 % that runs differ by at d = 2e4.  With long lists
// walks wait for their accumulators in device memory: values of 31015 rows against 5612 centres, 40 of 321 features each, 40.9 ms with 4096 rows, 34.9
// with 1024, 30.1 with 512; 20000 x 20000, 100 of 1000 features, 298, 248 and 217
constexpr int64_t kFillLeast = 512;
inline int64_t fill_group(int64_t M, int64_t d, int64_t nnz_c)
{
    const double span = 64.0 * (double)M * (double)d / (double)(nnz_c > 0 ? nnz_c : 1);
    int64_t rows = 4096;
    while (rows > kFillLeast && (double)rows > span) rows /= 2;
    return rows;
}
constexpr int kHashBits = 9;        // slots (2^9) of a wavefront's accumulator table in LDS
constexpr int kHashSlots = 1 << kHashBits;
constexpr int kHashMaxPairs = 320; // a row with at most this many pair updates uses the table (load <= 5/8)
// Where an input is swept more than once, the pairs and their K_ij - a_i b_j are written down before the first sweep and read
// by all of them, up to this many (8 bytes each); beyond it, and where there is no room, every sweep walks.  A walk adds
// into its accumulators at random, which is what it waits for; a reader streams.  200k rows of 100 entries against 20000
// centres: 1.19 ms by rows and 1.25 ms by columns walked; 1.16 ms to form the pairs, 0.075 ms and 0.046 ms
// read, so that two sweeps already gain (a product 5.72 -> 4.55 ms).  A fit of 21 sweeps, 100k rows and 10000 centres: 50.2 -> 41.3 ms.
constexpr unsigned long long kMaxPairs = (unsigned long long)1 << 29;
constexpr int kSide = 2;            // entries of X per lane that are looked up side by side
constexpr int kMaxHead = 128;       // features treated densely, at most (one dense row of X^H and C^H each)

// Passes over the rows of a CSR matrix: 16 lanes per row, so that a row's entries are read together (a thread per row read
// its 100 entries one after the other: 0.4 ms for the ids and 0.35 ms for the values of 200k rows, which are 0.16 and 0.08 GB)
constexpr int kRowLanes = 16;
constexpr int kRowSide = 4; // loads of a lane under way together
constexpr int64_t kRowPassBlocks = 16384; // workgroups of such a pass at most; each walks on
inline dim3 row_pass_grid(int64_t rows)
{
    const int64_t blocks = (rows + 256 / kRowLanes - 1) / (256 / kRowLanes);
    return dim3((unsigned)(blocks < kRowPassBlocks ? blocks : kRowPassBlocks));
}

// flag |= 1 if the CSR structure is not usable: indptr not starting at 0, decreasing, running
// past nnz, or the column indices of a row not strictly increasing inside [0, d)
__global__ __launch_bounds__(256) void csr_check_kernel(const int64_t *__restrict__ indptr, const int64_t *__restrict__ indices,
                                                       int64_t rows, int64_t nnz, int64_t d, int *flag)
{
    const int l = threadIdx.x % kRowLanes;
    bool bad = false;
    for (int64_t r = (int64_t)blockIdx.x * (256 / kRowLanes) + threadIdx.x / kRowLanes; r < rows;
         r += (int64_t)gridDim.x * (256 / kRowLanes)) {
        const int64_t p0 = indptr[r], p1 = indptr[r + 1];
        if ((r == 0 && p0 != 0) || p0 < 0 || p1 < p0 || p1 > nnz) {
            bad = true;
            continue; // its ids are not read
        }
        for (int64_t p = p0 + l; p < p1; p += kRowSide * kRowLanes) {
            int64_t c[kRowSide], prev[kRowSide];
#pragma unroll
            for (int u = 0; u < kRowSide; ++u) { // (past the end the row's last entry again)
                const int64_t e = p + u * kRowLanes < p1 ? p + u * kRowLanes : p1 - 1;
                c[u] = indices[e];
                prev[u] = indices[e > p0 ? e - 1 : e];
                if (e == p0) prev[u] = -1;
            }
#pragma unroll
            for (int u = 0; u < kRowSide; ++u)
                if (c[u] <= prev[u] || c[u] >= d) bad = true; // strictly increasing: every feature at most once in a row
        }
    }
    if (bad) atomicOr(flag, 1);
}

__global__ __launch_bounds__(256) void row_norms_kernel(const int64_t *__restrict__ indptr, const float *__restrict__ values,
                                                       int64_t rows, float *__restrict__ norms)
{
    const int l = threadIdx.x % kRowLanes;
    for (int64_t r = (int64_t)blockIdx.x * (256 / kRowLanes) + threadIdx.x / kRowLanes; r < rows;
         r += (int64_t)gridDim.x * (256 / kRowLanes)) {
        const int64_t p1 = indptr[r + 1];
        double s = 0.0;
        for (int64_t p = indptr[r] + l; p < p1; p += kRowSide * kRowLanes) {
            float v[kRowSide];
#pragma unroll
            for (int u = 0; u < kRowSide; ++u) v[u] = values[p + u * kRowLanes < p1 ? p + u * kRowLanes : p1 - 1];
#pragma unroll
            for (int u = 0; u < kRowSide; ++u) s += p + u * kRowLanes < p1 ? (double)v[u] * (double)v[u] : 0.0;
        }
#pragma unroll
        for (int w = kRowLanes / 2; w > 0; w >>= 1) s += __shfl_xor(s, w);
        if (l == 0) norms[r] = (float)s;
    }
}

// Where the feature ids reach far beyond the number of entries of the centres, the features that occur in a centre are
// numbered in the order of their ids and all lists go by that number: a word per 32 ids (which of them occur, how many do
// before them) takes the place of counters for all d, whose clearing, sums and search took 0.5 ms of a 4.5 ms product at
// d = 6.5e7.  Products with counters and with numbers: 20000 rows, 300 centres of 20 entries: d = 2e6 418 and 423 us, 4e6 412
// and 407, 6.4e7 684 and 376; 100k rows, 2000 centres of 100: d = 1e6 1530 and 1534 us, 4e6 1332 and 1277, 6.4e7 1232 and
// 871; 200k rows, 20000 centres of 100: d = 8e6 6.28 and 6.33 ms, 1.6e7 4.35 and 4.30, 6.4e7 4.30 and 3.91.
struct FeatureWord {
    unsigned bits;
    int before;
};
constexpr int64_t kRankedFrom = (int64_t)1 << 22;
inline bool ranked_features(int64_t d, int64_t nnz_c) { return d >= kRankedFrom && d / 8 >= nnz_c; }

// number of feature f: its id (words null), or its place among those that occur in a centre, -1 for one that does not
__device__ __forceinline__ int number_in(FeatureWord w, int64_t f)
{
    const unsigned bit = 1u << (f & 31);
    return (w.bits & bit) != 0 ? w.before + __popc(w.bits & (bit - 1u)) : -1;
}
__device__ __forceinline__ int feature_number(const FeatureWord *__restrict__ words, int64_t f)
{
    return words == nullptr ? (int)f : number_in(words[f >> 5], f);
}

// (a byte per id and plain stores: setting the bits took 2 M atomic operations, 168 us against 40 and a pass over the bytes)
__global__ void mark_features_kernel(const int64_t *__restrict__ indices, int64_t nnz, unsigned char *__restrict__ seen)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < nnz) seen[indices[p]] = 1;
}

// bits of the words from their 32 bytes, and how many each has
__global__ void word_counts_kernel(const uint4 *__restrict__ seen, int64_t len, FeatureWord *__restrict__ words, int *__restrict__ count)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= len) return;
    const uint4 lo = seen[2 * i], hi = seen[2 * i + 1];
    const unsigned part[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    unsigned bits = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) // (a byte is 0 or 1: the four of a part to its top nibble)
        bits |= ((part[k] * 0x10204080u) >> 28) << (4 * k);
    words[i].bits = bits;
    count[i] = __popc(bits);
}

// before <- the prefix sums of the counts, of which `local` are those inside a chunk and `sums` the chunks' own
__global__ void word_bases_kernel(const int *__restrict__ local, const int *__restrict__ sums, int64_t len,
                                  FeatureWord *__restrict__ words)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < len) words[i].before = local[i] + sums[i / kScanChunk];
}

// Number and row of every entry of the rows [row0, row1) of C, its place in its feature's list, and the lists' lengths: a wavefront per
// row.  Launched for one group of rows after the other, so that a feature's centre list
// comes out ordered by group: neighbouring list entries then update neighbouring accumulator
// entries (the same cache lines) when a long list is walked.  (Counting all entries first and taking the places
// in a second pass of atomics took 0.14 + 0.19 ms for 2 M entries and the row pointers on the host; 0.17 + 0.09 for csc_fill_kernel now.)
__global__ __launch_bounds__(256) void centre_entries_kernel(const int64_t *__restrict__ indptr, const int64_t *__restrict__ indices,
                                                            int64_t row0, int64_t row1, const FeatureWord *__restrict__ words,
                                                            int *__restrict__ number, int *__restrict__ row, int *__restrict__ place,
                                                            int *__restrict__ count)
{
    const int64_t r = row0 + (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= row1) return;
    const int64_t p1 = indptr[r + 1];
    for (int64_t p = indptr[r] + (threadIdx.x & 63); p < p1; p += 64) {
        const int f = feature_number(words, indices[p]);
        number[p] = f;
        row[p] = (int)r;
        place[p] = atomicAdd(&count[f], 1);
    }
}

// exclusive prefix sum of `in` (len entries) in three passes; out may alias in
__global__ __launch_bounds__(256) void scan_local_kernel(const int *__restrict__ in, int64_t len, int *__restrict__ out,
                                                        int *__restrict__ sums)
{
    __shared__ int sh[256];
    constexpr int kPer = kScanChunk / 256;
    const int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kPer;
    int v[kPer];
    int tot = 0;
    if (base + kPer <= len) { // (the arrays are allocated: a thread's entries are 64-byte aligned)
        int4 x[kPer / 4];
#pragma unroll
        for (int e = 0; e < kPer / 4; ++e) x[e] = reinterpret_cast<const int4 *>(in + base)[e];
#pragma unroll
        for (int e = 0; e < kPer / 4; ++e) {
            v[4 * e] = x[e].x;
            v[4 * e + 1] = x[e].y;
            v[4 * e + 2] = x[e].z;
            v[4 * e + 3] = x[e].w;
        }
    } else {
#pragma unroll
        for (int e = 0; e < kPer; ++e) v[e] = (base + e < len) ? in[base + e] : 0;
    }
#pragma unroll
    for (int e = 0; e < kPer; ++e) tot += v[e];
    sh[threadIdx.x] = tot;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        const int add = ((int)threadIdx.x >= off) ? sh[threadIdx.x - off] : 0;
        __syncthreads();
        sh[threadIdx.x] += add;
        __syncthreads();
    }
    int run = sh[threadIdx.x] - tot; // exclusive prefix of this thread inside the workgroup
    if (base + kPer <= len) {
#pragma unroll
        for (int e = 0; e < kPer / 4; ++e) {
            int4 x;
            x.x = run;
            x.y = x.x + v[4 * e];
            x.z = x.y + v[4 * e + 1];
            x.w = x.z + v[4 * e + 2];
            run = x.w + v[4 * e + 3];
            reinterpret_cast<int4 *>(out + base)[e] = x;
        }
    } else {
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
            if (base + e < len) out[base + e] = run;
            run += v[e];
        }
    }
    if (threadIdx.x == 255) sums[blockIdx.x] = sh[255];
}

__global__ __launch_bounds__(256) void scan_sums_kernel(int *__restrict__ sums, int64_t count)
{
    __shared__ int sh[256];
    const int64_t per = (count + 255) / 256;
    const int64_t b0 = (int64_t)threadIdx.x * per;
    int tot = 0;
    for (int64_t i = b0; i < b0 + per && i < count; ++i) tot += sums[i];
    sh[threadIdx.x] = tot;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        const int add = ((int)threadIdx.x >= off) ? sh[threadIdx.x - off] : 0;
        __syncthreads();
        sh[threadIdx.x] += add;
        __syncthreads();
    }
    int run = sh[threadIdx.x] - tot;
    for (int64_t i = b0; i < b0 + per && i < count; ++i) {
        const int v = sums[i];
        sums[i] = run;
        run += v;
    }
}

__global__ void scan_add_kernel(int *__restrict__ out, int64_t len, const int *__restrict__ sums)
{
    const int64_t i = 4 * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x); // kScanChunk is a multiple of 4
    if (i >= len) return;
    const int add = sums[i / kScanChunk];
    if (i + 3 < len) {
        int4 x = *reinterpret_cast<const int4 *>(out + i);
        x.x += add;
        x.y += add;
        x.z += add;
        x.w += add;
        *reinterpret_cast<int4 *>(out + i) = x;
    } else {
        for (int64_t k = i; k < len; ++k) out[k] += add;
    }
}

// the CSC image of C from the entries' numbers and places
__global__ void csc_fill_kernel(const int *__restrict__ number, const int *__restrict__ place, const int *__restrict__ row,
                                const float *__restrict__ values, int64_t nnz, const int *__restrict__ col_ptr,
                                int *__restrict__ csc_row, float *__restrict__ csc_val)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= nnz) return;
    const int pos = col_ptr[number[p]] + place[p];
    csc_row[pos] = row[p];
    csc_val[pos] = values[p];
}

// e[r] = exp(-norm[r] / 2 sigma^2)
__global__ void norm_factor_kernel(const float *__restrict__ norms, int64_t rows, float inv2s2, float *__restrict__ e)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r < rows) e[r] = expf(-norms[r] * inv2s2);
}

// partial sums of e[r] * vec[r * ldv] in fp64, fixed order: one partial per workgroup
__global__ __launch_bounds__(256) void weighted_sum_kernel(const float *__restrict__ e, const float *__restrict__ vec,
                                                          int64_t ldv, int64_t rows, double *__restrict__ part)
{
    __shared__ double sh[256];
    double s = 0.0;
    for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < rows; r += (int64_t)gridDim.x * 256)
        s += (double)e[r] * (double)vec[r * ldv];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// Column sweep: the all-pairs part of U in fp64, base[j] = e[j] * s (rank-one form, x null) or
// e[j] * x[j] (dense head product).  The sparse walk scatters its terms into a separate fp64
// buffer and the two are added at the end: float atomics onto the all-pairs part, which is
// orders of magnitude larger than a single term, would lose the terms' low bits at every add.
__global__ void column_base_kernel(const float *__restrict__ e, const float *__restrict__ x, double s, int64_t rows,
                                   double *__restrict__ base)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r < rows) base[r] = (double)e[r] * (x ? (double)x[r] : s);
}

// out[j * ldo] = base[j] + scattered[j]
__global__ void column_finish_kernel(const double *__restrict__ base, const double *__restrict__ scattered, int64_t rows,
                                     float *__restrict__ out, int64_t ldo)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r < rows) out[r * ldo] = (float)(base[r] + scattered[r]);
}

// Orders a wavefront's accesses to its private accumulator: everything it has issued (atomics
// without a return value included) has been performed at the L2, where all accesses to the
// accumulator take place, before anything that follows.  A workgroup-scope fence is that wait and
// nothing else; a device-scope one would also write back and invalidate the XCD's whole L2 at every
// row, which evicts the accumulator lines the next pass is about to hit.
__device__ __forceinline__ void accumulator_fence() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup"); }

// ---- head features ---------------------------------------------------------------------
//
// A feature that occurs in a large share of the centres (and hence of the rows) makes nearly every
// pair of points share a feature: its centre list is long and is walked for every row that has
// the feature, and a handful of such features carry most of the pair updates.  They are taken out
// of the sparse walk and treated densely instead.  With H the set of head features, x^H / c^H the
// dense head parts of the points and g = g^H + g^T split accordingly,
//   K_ij = KH_ij + KH_ij (exp(g^T_ij / sigma^2) - 1),    KH_ij = a_i b_j exp(g^H_ij / sigma^2),
// the first term over all pairs and the second only over pairs that share a tail feature.  KH is
// the Gaussian kernel of the head parts times the factors a^T_i = exp(-|x^T_i|^2 / 2 sigma^2) and
// b^T_j of the tail parts' norms, so its sweep is one dense product with d = |H| on the dense
// engines; the second term is the sparse walk over the tail features, whose pairs read g^H from
// the dense head rows of the few head features their row has.

// features whose centre list has at least min_len entries: (feature, list start, length)
__global__ void head_candidates_kernel(const int *__restrict__ col_ptr, int64_t d, int min_len, int cap,
                                       int *__restrict__ count, int *__restrict__ cand)
{
    const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= d) return;
    const int q0 = col_ptr[f], len = col_ptr[f + 1] - q0;
    if (len < min_len) return;
    const int at = atomicAdd(count, 1);
    if (at < cap) {
        cand[3 * at] = (int)f;
        cand[3 * at + 1] = q0;
        cand[3 * at + 2] = len;
    }
}

struct HeadLists {
    int q0[kMaxHead], len[kMaxHead];
};

// CH[j, h] = c_j's value of head feature h (CH zeroed before); blockIdx.y = h
__global__ void head_centres_kernel(HeadLists hl, int Hn, const int *__restrict__ csc_row,
                                    const float *__restrict__ csc_val, float *__restrict__ CH)
{
    const int h = blockIdx.y;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < hl.len[h]) CH[(int64_t)csc_row[hl.q0[h] + k] * Hn + h] = csc_val[hl.q0[h] + k];
}

// e[r] = exp(-(norm[r] - |row r of PH|^2) / 2 sigma^2): the factor of the tail part's norm; *worst =
// bits of the largest |row of PH|^2 / 2 sigma^2 (non-negative floats order like their bit patterns)
__global__ void tail_factor_kernel(const float *__restrict__ norms, const float *__restrict__ PH, int Hn, int64_t rows,
                                   float inv2s2, float *__restrict__ e, unsigned *__restrict__ worst)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    float hn = 0.0f;
    if (r < rows) {
#pragma unroll 4
        for (int h = 0; h < Hn; ++h) hn = fmaf(PH[r * Hn + h], PH[r * Hn + h], hn);
        e[r] = expf(-fmaxf(norms[r] - hn, 0.0f) * inv2s2);
    }
    // (one atomic per wavefront, and only where it can raise the maximum: with one per row the two launches of 200k and 20000 rows
    // took 56 us, 39 now)
    unsigned most = __float_as_uint(hn * inv2s2);
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) most = max(most, (unsigned)__shfl_xor((int)most, w));
    if ((threadIdx.x & 63) == 0 && most > __hip_atomic_load(worst, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(worst, most);
}

// out[r * ldo] = e[r] * x[r * ldx]
__global__ void scale_kernel(const float *__restrict__ e, const float *__restrict__ x, int64_t ldx, int64_t rows,
                             float *__restrict__ out, int64_t ldo)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r < rows) out[r * ldo] = e[r] * x[r * ldx];
}

// The number of pairs is added up in several words, a cache line each: one atomic per wavefront on a single word made the work list of
// 17223 rows of 13 entries 103 us, 7 without
constexpr int kTotals = 15, kTotalStride = 16;

// Work list of X (see SparseArgs): one wavefront per row looks every entry's feature up in the
// centre lists once, so that the sweeps stream (start, length, value) instead of reading the
// list pointers at random for every entry, pass and sweep; entries whose feature occurs in no
// centre drop out.  Entries of head features (head_feat: Hn ids, ascending) go to the back of
// the row's range as (head index, value) and into the dense row XH[row, :] (zeroed before).
__global__ __launch_bounds__(kSpThreads) void build_work_kernel(const int64_t *__restrict__ x_indptr,
                                                               const int64_t *__restrict__ x_indices,
                                                               const float *__restrict__ x_values, int64_t n,
                                                               const FeatureWord *__restrict__ words, const int *__restrict__ col_ptr,
                                                               const int *__restrict__ head_feat, int Hn, int head_min_len,
                                                               int *__restrict__ work_count, int *__restrict__ work_pairs,
                                                               int *__restrict__ head_count,
                                                               int *__restrict__ work_q0, int *__restrict__ work_len,
                                                               float *__restrict__ work_val, float *__restrict__ XH,
                                                               int64_t M, int *__restrict__ pair_cap,
                                                               unsigned long long *__restrict__ pair_totals)
{
    const int lane = threadIdx.x & 63;
    const int64_t wave = (int64_t)blockIdx.x * kSpWaves + (threadIdx.x >> 6);
    const int64_t waves = (int64_t)gridDim.x * kSpWaves;
    __shared__ int heads_of[kMaxHead];
    __shared__ unsigned long long totals[kSpWaves];
    if ((int)threadIdx.x < Hn) heads_of[threadIdx.x] = head_feat[threadIdx.x];
    __syncthreads();
    const unsigned long long below = (1ull << lane) - 1ull;
    unsigned long long total = 0;
    int64_t next0 = 0, next1 = 0; // range of the next row
    if (wave < n) {
        next0 = x_indptr[wave];
        next1 = x_indptr[wave + 1];
    }
    for (int64_t row = wave; row < n; row += waves) {
        const int64_t p0 = next0, p1 = next1;
        if (row + waves < n) {
            next0 = x_indptr[row + waves];
            next1 = x_indptr[row + waves + 1];
        }
        int64_t kept = 0, heads = 0, pairs = 0;
        // An entry is a chain of three loads (id, word, list), so a lane takes kSide entries at a time, past the end its row's
        // last one again: no load waits behind a branch
        for (int64_t p = p0; p < p1; p += 64 * kSide) {
            int64_t id[kSide];
            float xv[kSide];
            int f[kSide], q0[kSide], len[kSide], h[kSide];
            FeatureWord w[kSide];
#pragma unroll
            for (int u = 0; u < kSide; ++u) {
                const int64_t e = p + 64 * u + lane < p1 ? p + 64 * u + lane : p1 - 1;
                id[u] = x_indices[e];
                xv[u] = x_values[e];
            }
            if (words != nullptr) {
#pragma unroll
                for (int u = 0; u < kSide; ++u) w[u] = words[id[u] >> 5];
#pragma unroll
                for (int u = 0; u < kSide; ++u) f[u] = number_in(w[u], id[u]);
            } else {
#pragma unroll
                for (int u = 0; u < kSide; ++u) f[u] = (int)id[u];
            }
#pragma unroll
            for (int u = 0; u < kSide; ++u) {
                if (p + 64 * u + lane >= p1) f[u] = -1;
                const int at = f[u] < 0 ? 0 : f[u];
                q0[u] = col_ptr[at];
                len[u] = col_ptr[at + 1];
            }
#pragma unroll
            for (int u = 0; u < kSide; ++u) {
                len[u] = f[u] < 0 ? 0 : len[u] - q0[u];
                h[u] = -1;
                if (Hn > 0 && len[u] >= head_min_len) { // binary search among the head features
                    int lo = 0, hi = Hn - 1;
                    while (lo < hi) {
                        const int mid = (lo + hi) >> 1;
                        if (heads_of[mid] < f[u]) lo = mid + 1;
                        else hi = mid;
                    }
                    if (heads_of[lo] == f[u]) h[u] = lo;
                }
            }
#pragma unroll
            for (int u = 0; u < kSide; ++u) {
                const bool tail = len[u] > 0 && h[u] < 0;
                const unsigned long long keep = __ballot(tail);
                const unsigned long long head = __ballot(h[u] >= 0);
                if (tail) {
                    const int64_t at = p0 + kept + __popcll(keep & below);
                    work_q0[at] = q0[u];
                    work_len[at] = len[u];
                    work_val[at] = xv[u];
                }
                if (h[u] >= 0) {
                    const int64_t at = p1 - 1 - heads - __popcll(head & below);
                    work_q0[at] = h[u];
                    work_val[at] = xv[u];
                    XH[row * Hn + h[u]] = xv[u];
                }
                kept += __popcll(keep);
                heads += __popcll(head);
                pairs += tail ? len[u] : 0;
            }
        }
        for (int w = 32; w > 0; w >>= 1) pairs += __shfl_xor(pairs, w);
        if (lane == 0) {
            work_count[row] = (int)kept;
            work_pairs[row] = (int)(pairs < 0x7fffffffLL ? pairs : 0x7fffffffLL);
            head_count[row] = (int)heads;
            pair_cap[row] = (int)(pairs < M ? pairs : M);
        }
        total += (unsigned long long)(pairs < M ? pairs : M);
    }
    if (pair_totals == nullptr) return; // (the same for all)
    if (lane == 0) totals[threadIdx.x >> 6] = total;
    __syncthreads();
    if (threadIdx.x == 0) {
        total = 0;
        for (int w = 0; w < kSpWaves; ++w) total += totals[w];
        if (total > 0) atomicAdd(pair_totals + blockIdx.x % kTotals * kTotalStride, total);
    }
}

// A pair of points that share a tail feature: the centre and K_ij - KH_ij
struct SparsePair {
    int centre;
    float excess;
};

struct SparseArgs {
    const int64_t *x_indptr;
    // work list of X: per row the entries whose feature occurs in some centre, packed to the front
    // of the row's own range [x_indptr[r], x_indptr[r] + work_count[r]): start and length of the
    // feature's centre list and the entry's value
    const int *work_count, *work_q0, *work_len;
    const float *work_val;
    const int *work_pairs; // per row: sum of the list lengths of its work list (saturating)
    // head features (Hn = 0: none): per row the last head_count[r] slots of its range hold (head
    // index, value); CH is the dense M x Hn image of the centres' head parts; tail_factor the
    // factor a^T of the rows (row sweep); dense the head-kernel product of the row sweep
    int Hn;
    const int *head_count;
    const float *CH, *tail_factor, *dense;
    int64_t n, M;
    const int *csc_row;
    const float *csc_val;
    const float *xn, *cn; // squared norms
    const float *xa;      // a_i
    const float *vec;     // row sweep: v over the centres; column sweep: w over the rows
    int64_t ldv;
    float *out;           // row sweep: W over the rows
    double *scattered;    // column sweep: the walk's terms of U over the centres (zero before)
    int64_t ldo;
    float *acc;           // one dense accumulator of M floats per wavefront of the grid
    float inv2s2, inv_s2;
    double s_rank_one;    // row sweep: sum_j b_j v_j
    // pair lists: those of row r start at pairs[pair_off[r]], pair_count[r] of them
    const int *pair_off;
    int *pair_count;
    SparsePair *pairs;
};

// K_ij - KH_ij from the tail part gt and the head part gh of the dot product and the squared norms
// (no head features: gh = 0 and KH_ij = a_i b_j).  With e0 = -log KH_ij >= 0 and a = gt / sigma^2 the
// excess is exp(a - e0) - exp(-e0), where a - e0 = log K_ij <= 0: neither term can overflow.  For
// small a the difference is taken as exp(-e0) expm1(a), which keeps its leading digits.
__device__ __forceinline__ float pair_excess(float gt, float gh, float xn, float cn, float inv2s2, float inv_s2)
{
    const float e0 = (xn + cn) * inv2s2 - gh * inv_s2;
    const float a = gt * inv_s2;
    if (a < 1.0f) return expf(-e0) * expm1f(a);
    return expf(a - e0) - expf(-e0);
}

// Adds v to the entry of key j of a wavefront's table (open addressing, linear probing; the
// table never holds more than kHashMaxPairs keys, so a free slot is always found); a new key's slot goes to `used`
__device__ __forceinline__ void table_add(int *keys, float *vals, unsigned short *used, int *count, int j, float v)
{
    unsigned slot = ((unsigned)j * 2654435761u) >> (32 - kHashBits);
    for (;;) {
        const int prev = atomicCAS(&keys[slot], -1, j);
        if (prev == -1) used[atomicAdd(count, 1)] = (unsigned short)slot;
        if (prev == -1 || prev == j) {
            unsafeAtomicAdd(&vals[slot], v);
            return;
        }
        slot = (slot + 1) & (kHashSlots - 1);
    }
}

// A wavefront's own LDS accesses, in order
__device__ __forceinline__ void lds_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local"); }

// The updates of a row, 64 at a time, one per lane, whatever the lengths of its lists: the lists of 64 entries (entry(p, q0, len, x):
// start and length, > 0, of its list, and its value) are laid end to end, the places where they start are marked in a word, and
// the marks up to a lane count its list.  visit(q, x) for place q of a list.  With a list of up to 31 per lane, and the whole wavefront
// for longer ones, a row of 12 lists and 50 updates, the usual case, kept 12 lanes busy for the longest: forming the
// pairs of 200k rows and 20000 centres took 1.16 ms, 0.65 now (with the table read through the list of its slots, not searched).
template <class T, class Entry, class Visit>
__device__ __forceinline__ void walk_lists(int64_t p0, int64_t p1, int lane, unsigned long long *starts, Entry &&entry, Visit &&visit)
{
    for (int64_t p = p0; p < p1; p += 64) {
        const bool mine = p + lane < p1;
        int q0 = 0, len = 0;
        T xv = 0;
        if (mine) entry(p + lane, q0, len, xv);
        int end = len;
#pragma unroll
        for (int w = 1; w < 64; w <<= 1) {
            const int o = __shfl_up(end, w);
            if (lane >= w) end += o;
        }
        const int start = end - len, total = __shfl(end, 63);
        for (int k0 = 0; k0 < total; k0 += 64) {
            if (lane == 0) *starts = 0;
            lds_order();
            if (mine && start >= k0 && start < k0 + 64) atomicOr(starts, 1ull << (start - k0));
            lds_order();
            const unsigned long long marks = *starts;
            const int from = __popcll(__ballot(mine && start < k0)) + __popcll(marks & (~0ull >> (63 - lane))) - 1;
            const int q = __shfl(q0 - start, from) + k0 + lane;
            const T x = __shfl(xv, from);
            if (k0 + lane < total) visit(q, x);
            lds_order();
        }
    }
}

enum SparseMode { kRowSweep, kColumnSweep, kFormPairs };
// (kFormPairs: the pairs are written down, for sweeps that read them)
template <SparseMode MODE>
__global__ __launch_bounds__(kSpThreads) void sparse_sweep_kernel(SparseArgs a)
{
    const int lane = threadIdx.x & 63;
    const int64_t wave = (int64_t)blockIdx.x * kSpWaves + (threadIdx.x >> 6);
    const int64_t waves = (int64_t)gridDim.x * kSpWaves;
    float *acc = a.acc + wave * a.M;
    // the head features of the row in hand, for every lane of the wavefront to read
    __shared__ int head_idx_all[kSpWaves][kMaxHead];
    __shared__ float head_val_all[kSpWaves][kMaxHead];
    int *const head_idx = head_idx_all[threadIdx.x >> 6];
    float *const head_val = head_val_all[threadIdx.x >> 6];
    // Rows with few pair updates accumulate in a table in LDS instead of the dense accumulator in
    // device memory: (centre, sum) pairs, all slots empty (key -1, sum 0) between rows.
    __shared__ int keys_all[kSpWaves][kHashSlots];
    __shared__ float vals_all[kSpWaves][kHashSlots];
    int *const keys = keys_all[threadIdx.x >> 6];
    float *const vals = vals_all[threadIdx.x >> 6];
    __shared__ int formed_all[kSpWaves]; // pairs of the row in hand: taken slots of the table, or those written down
    __shared__ unsigned short used_all[kSpWaves][kHashMaxPairs]; // the slots
    __shared__ unsigned long long starts_all[kSpWaves];
    int *const formed = &formed_all[threadIdx.x >> 6];
    unsigned short *const used = used_all[threadIdx.x >> 6];
    unsigned long long *const starts = &starts_all[threadIdx.x >> 6];
    if (lane == 0) *formed = 0;
    for (int k = lane; k < kHashSlots; k += 64) {
        keys[k] = -1;
        vals[k] = 0.0f;
    }
    accumulator_fence();
    bool cleared = false;
    for (int64_t row = wave; row < a.n; row += waves) {
        const int64_t p0 = a.x_indptr[row], p1 = p0 + a.work_count[row];
        const float xn = a.xn[row];
        const float wrow = MODE == kColumnSweep ? a.vec[row * a.ldv] : 0.0f;
        SparsePair *const list = MODE == kFormPairs ? a.pairs + a.pair_off[row] : nullptr;
        const bool in_lds = a.work_pairs[row] <= kHashMaxPairs; // same for the whole wavefront
        float sum = 0.0f;
        int hc = 0;
        if (a.Hn > 0) {
            hc = a.head_count[row];
            const int64_t back = a.x_indptr[row + 1] - hc;
            for (int k = lane; k < hc; k += 64) { // hc <= Hn <= kMaxHead, which may exceed the 64 lanes
                head_idx[k] = a.work_q0[back + k];
                head_val[k] = a.work_val[back + k];
            }
            accumulator_fence(); // the wavefront's own LDS writes, before any lane reads them
        }
        // g^H_ij of the row in hand against centre j
        auto head_dot = [&](int j) -> float {
            float gh = 0.0f;
#pragma unroll 4
            for (int k = 0; k < hc; ++k) gh = fmaf(head_val[k], a.CH[(int64_t)j * a.Hn + head_idx[k]], gh);
            return gh;
        };
        // one term x_if c_jf of g^T_ij
        auto add = [&](int j, float v) {
            if (in_lds) table_add(keys, vals, used, formed, j, v);
            else unsafeAtomicAdd(&acc[j], v);
        };
        // the finished g^T_ij of a pair that shares a tail feature, the k-th of the row
        auto consume = [&](int j, float g, int k) {
            const float ex = pair_excess(g, head_dot(j), xn, a.cn[j], a.inv2s2, a.inv_s2);
            if (MODE == kColumnSweep) unsafeAtomicAdd(&a.scattered[j], (double)ex * (double)wrow);
            else if (MODE == kRowSweep) sum += ex * a.vec[j * a.ldv];
            else list[k] = {j, ex}; // (each centre at most once, so no more than the row has room for)
        };
        auto walk = [&](auto &&visit) {
            walk_lists<float>(p0, p1, lane, starts, [&](int64_t p, int &q0, int &len, float &x) {
                q0 = a.work_q0[p];
                len = a.work_len[p];
                x = a.work_val[p];
            }, visit);
            accumulator_fence(); // every lane's updates are done before what follows
        };
        // The accumulator in device memory is cleared by its first row: few rows of a usual input need one, and clearing all of
        // them ahead (0.66 GB at M = 20000) took 0.11 ms of a 3.5 ms product.  Every row leaves it zero.
        if (!in_lds && !cleared) {
            for (int64_t j = lane; j < a.M; j += 64) __hip_atomic_store(&acc[j], 0.0f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            accumulator_fence();
            cleared = true;
        }
        // x_if c_jf goes into the accumulator, then every touched entry is taken out again: in LDS through the list of the
        // table's slots, in device memory by walking the lists a second time (atomic exchange with zero, so a
        // centre reached through several features is consumed once)
        walk([&](int q, float x) { add(a.csc_row[q], x * a.csc_val[q]); });
        if (in_lds) {
            const int count = *formed;
            for (int k = lane; k < count; k += 64) {
                const int slot = used[k];
                const int j = keys[slot];
                const float g = vals[slot];
                keys[slot] = -1;
                vals[slot] = 0.0f;
                consume(j, g, k);
            }
        } else {
            walk([&](int q, float) {
                const int j = a.csc_row[q];
                const float g = atomicExch(&acc[j], 0.0f);
                if (g != 0.0f) consume(j, g, MODE == kFormPairs ? atomicAdd(formed, 1) : 0); // (or it was taken out before)
            });
        }
        accumulator_fence();
        if (lane == 0) {
            if (MODE == kFormPairs) a.pair_count[row] = *formed;
            *formed = 0;
        }
        accumulator_fence();
        if (MODE == kRowSweep) {
            sum += __shfl_xor(sum, 32);
            sum += __shfl_xor(sum, 16);
            sum += __shfl_xor(sum, 8);
            sum += __shfl_xor(sum, 4);
            sum += __shfl_xor(sum, 2);
            sum += __shfl_xor(sum, 1);
            if (lane == 0) {
                const float all_pairs = a.Hn > 0 ? a.tail_factor[row] * a.dense[row] : (float)((double)a.xa[row] * a.s_rank_one);
                a.out[row * a.ldo] = all_pairs + sum;
            }
        }
    }
}

// The sweeps over pair lists: 16 lanes per row, sums in fp64.
__global__ __launch_bounds__(256) void pair_rows_kernel(SparseArgs a)
{
    const int l = threadIdx.x % kRowLanes;
    for (int64_t r = (int64_t)blockIdx.x * (256 / kRowLanes) + threadIdx.x / kRowLanes; r < a.n; r += (int64_t)gridDim.x * (256 / kRowLanes)) {
        const SparsePair *const list = a.pairs + a.pair_off[r];
        const int count = a.pair_count[r];
        double s = 0.0;
        for (int k = l; k < count; k += 4 * kRowLanes) {
            SparsePair p[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) p[u] = list[k + u * kRowLanes < count ? k + u * kRowLanes : k];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                s += k + u * kRowLanes < count ? (double)p[u].excess * (double)a.vec[(int64_t)p[u].centre * a.ldv] : 0.0;
        }
#pragma unroll
        for (int w = kRowLanes / 2; w > 0; w >>= 1) s += __shfl_xor(s, w);
        if (l == 0) {
            const float all_pairs = a.Hn > 0 ? a.tail_factor[r] * a.dense[r] : (float)((double)a.xa[r] * a.s_rank_one);
            a.out[r * a.ldo] = (float)((double)all_pairs + s);
        }
    }
}
// A workgroup has a range of `width` centres in LDS, one fp64 sum each (20480 fill the 160 KB), and adds up the pairs of its share of the rows
// there; the workgroups' sums are merged.  (fp64 atomics in device memory took
// 0.605 ms for 200k rows against 20000 centres, 0.046 ms this way.)  Every range of centres reads all pairs; products with walks and with
// pairs, rows of 100 entries: 100k x 30000 (2 ranges) 3.04 and 2.46 ms, 100k x 60000 (3) 7.04 and 5.27, 200k x 100k (5) 20.5 and 14.4, 200k x
// 200k (10) 44.9 and 30.7, 330k x 327k (16) 123 and 83, 20000 x 327k (16) 20.4 and 14.9.
constexpr int kPairThreads = 1024;
constexpr int kPairWidth = 20480;
__global__ __launch_bounds__(kPairThreads) void pair_columns_kernel(SparseArgs a, int width, double *__restrict__ part)
{
    extern __shared__ __attribute__((aligned(16))) double sums[];
    const int lo = (int)blockIdx.y * width, here = (int)(a.M - lo < width ? a.M - lo : width);
    for (int j = threadIdx.x; j < here; j += kPairThreads) sums[j] = 0.0;
    __syncthreads();
    const int l = threadIdx.x % kRowLanes;
    constexpr int kGroups = kPairThreads / kRowLanes;
    for (int64_t r = (int64_t)blockIdx.x * kGroups + threadIdx.x / kRowLanes; r < a.n; r += (int64_t)gridDim.x * kGroups) {
        const SparsePair *const list = a.pairs + a.pair_off[r];
        const int count = a.pair_count[r];
        const double w = (double)a.vec[r * a.ldv];
        for (int k = l; k < count; k += 4 * kRowLanes) {
            SparsePair p[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) p[u] = list[k + u * kRowLanes < count ? k + u * kRowLanes : k];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int j = p[u].centre - lo;
                if (k + u * kRowLanes < count && j >= 0 && j < here) unsafeAtomicAdd(&sums[j], (double)p[u].excess * w);
            }
        }
    }
    __syncthreads();
    for (int j = threadIdx.x; j < here; j += kPairThreads) part[(int64_t)blockIdx.x * a.M + lo + j] = sums[j];
}

inline dim3 grid_for(int64_t n, int threads = 256) { return dim3((unsigned)((n + threads - 1) / threads)); }

// fp64 entries of the centres' kernel matrix, for the preconditioner: column i of the upper triangle
// (column-major K, leading dimension ldk) = exp(-(|c_i|^2 + |c_j|^2 - 2 g_ij) / 2 sigma^2) + jitter [i == j],
// j <= i, with g_ij accumulated in a private fp64 accumulator exactly as in the sweeps (every
// entry of the accumulator up to i is read and cleared when the column is written out).  A wavefront writes 64
// consecutive entries; along a row of K, ldk apart, 10000 centres took 1.40 ms, 0.49 now.
__global__ __launch_bounds__(kSpThreads) void sparse_kmm_kernel(const int64_t *__restrict__ c_indptr,
                                                               const int *__restrict__ number,
                                                               const float *__restrict__ c_values, int64_t M,
                                                               const int *__restrict__ col_ptr,
                                                               const int *__restrict__ csc_row,
                                                               const float *__restrict__ csc_val,
                                                               const double *__restrict__ cn, double inv2s2,
                                                               double jitter, double *__restrict__ acc_all,
                                                               double *__restrict__ K, int64_t ldk)
{
    const int lane = threadIdx.x & 63;
    const int64_t wave = (int64_t)blockIdx.x * kSpWaves + (threadIdx.x >> 6);
    const int64_t waves = (int64_t)gridDim.x * kSpWaves;
    double *acc = acc_all + wave * M;
    __shared__ unsigned long long starts_all[kSpWaves];
    unsigned long long *const starts = &starts_all[threadIdx.x >> 6];
    for (int64_t col = wave; col < M; col += waves) {
        walk_lists<double>(c_indptr[col], c_indptr[col + 1], lane, starts, [&](int64_t p, int &q0, int &len, double &x) {
            const int f = number[p];
            q0 = col_ptr[f];
            len = col_ptr[f + 1] - q0;
            x = (double)c_values[p];
        }, [&](int q, double x) {
            const int j = csc_row[q];
            if (j <= col) unsafeAtomicAdd(&acc[j], x * (double)csc_val[q]);
        });
        accumulator_fence();
        const double ci = cn[col];
        for (int64_t j = lane; j <= col; j += 64) {
            // written by atomics (at the L2): read and cleared there too, past the first-level cache
            const double g = __hip_atomic_load(&acc[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (g != 0.0) __hip_atomic_store(&acc[j], 0.0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            K[j + col * ldk] = exp(-(ci + cn[j] - 2.0 * g) * inv2s2) + (j == col ? jitter : 0.0);
        }
        accumulator_fence();
    }
}

__global__ void row_norms_f64_kernel(const int64_t *__restrict__ indptr, const float *__restrict__ values, int64_t rows,
                                     double *__restrict__ norms)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= rows) return;
    double s = 0.0;
    for (int64_t p = indptr[r]; p < indptr[r + 1]; ++p) s += (double)values[p] * (double)values[p];
    norms[r] = s;
}

// out[r] = w[r] * x[r * ldx]
__global__ void weigh_kernel(const float *__restrict__ x, int64_t ldx, const float *__restrict__ w, int64_t rows,
                             float *__restrict__ out)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r < rows) out[r] = w[r] * x[r * ldx];
}

// structure check of one CSR matrix before anything indexes with the caller's numbers; *nnz_out
// receives indptr[rows]
int check_csr(knm_ctx *ctx, const int64_t *indptr, const int64_t *indices, int64_t rows, int64_t d, int64_t *nnz_out)
{
    hipStream_t st = ctx->stream;
    int64_t nnz = 0;
    hipError_t e = hipMemcpyAsync(&nnz, indptr + rows, sizeof(int64_t), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "reading the CSR size", e);
    if (nnz < 0 || nnz >= 0x7fffffffLL * 64) return fail(ctx, KNM_INVALID_ARG, "bad CSR size");
    DevBuf flag;
    if (flag.alloc(ctx, sizeof(int)) != hipSuccess) return fail(ctx, KNM_ALLOC, "hipMalloc");
    int bad = 0;
    e = hipMemsetAsync(flag.p, 0, sizeof(int), st);
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipMemsetAsync", e);
    hipLaunchKernelGGL(csr_check_kernel, row_pass_grid(rows), dim3(256), 0, st, indptr, indices, rows, nnz, d, flag.as<int>());
    e = hipMemcpyAsync(&bad, flag.p, sizeof(int), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "CSR check", e);
    if (bad)
        return fail(ctx, KNM_INVALID_ARG,
                    "CSR structure: row pointers not monotone from 0, or feature ids of a row not strictly increasing in [0, d)");
    *nnz_out = nnz;
    return KNM_OK;
}

// CSC image of the centres: col_ptr (features + 1), csc_row / csc_val (nnz_c); `number` of every entry of C (CSR order)
struct CentreLists {
    DevBuf words, col_ptr, csc_row, csc_val, number;
    int64_t features = 0; // lists, empty ones included
    int build(knm_ctx *ctx, const int64_t *c_indptr, const int64_t *c_indices, const float *c_values, int64_t M,
              int64_t d, int64_t nnz_c)
    {
        hipStream_t st = ctx->stream;
        if (nnz_c >= 0x7fffffffLL) return fail(ctx, KNM_UNSUPPORTED, "more than 2^31 - 2 stored entries in C");
        DevBuf counts, sums, row, place, seen;
        const bool ranked = nnz_c > 0 && ranked_features(d, nnz_c);
        const int64_t n_words = (d + 31) / 32;
        features = ranked ? nnz_c : d; // (no more than occur)
        const int64_t scan_blocks = ((ranked && n_words > features + 1 ? n_words : features + 1) + kScanChunk - 1) / kScanChunk;
        const int64_t fill_blocks = (features + 1 + kScanChunk - 1) / kScanChunk;
        if (col_ptr.alloc(ctx, sizeof(int) * (features + 1)) != hipSuccess || sums.alloc(ctx, sizeof(int) * scan_blocks) != hipSuccess ||
            csc_row.alloc(ctx, sizeof(int) * nnz_c) != hipSuccess || csc_val.alloc(ctx, sizeof(float) * nnz_c) != hipSuccess ||
            number.alloc(ctx, sizeof(int) * nnz_c) != hipSuccess || row.alloc(ctx, sizeof(int) * nnz_c) != hipSuccess ||
            place.alloc(ctx, sizeof(int) * nnz_c) != hipSuccess || (ranked && counts.alloc(ctx, sizeof(int) * n_words) != hipSuccess) ||
            (ranked && (words.alloc(ctx, sizeof(FeatureWord) * n_words) != hipSuccess || seen.alloc(ctx, 32 * n_words) != hipSuccess))) {
            (void)hipGetLastError();
            return fail(ctx, KNM_ALLOC, "hipMalloc(centre lists)");
        }
        hipError_t e = hipMemsetAsync(col_ptr.p, 0, sizeof(int) * (features + 1), st);
        if (e == hipSuccess && ranked) e = hipMemsetAsync(seen.p, 0, 32 * n_words, st);
        if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipMemsetAsync", e);
        if (ranked) {
            const int64_t blocks = (n_words + kScanChunk - 1) / kScanChunk;
            hipLaunchKernelGGL(mark_features_kernel, grid_for(nnz_c), dim3(256), 0, st, c_indices, nnz_c, seen.as<unsigned char>());
            hipLaunchKernelGGL(word_counts_kernel, grid_for(n_words), dim3(256), 0, st, seen.as<uint4>(), n_words,
                               words.as<FeatureWord>(), counts.as<int>());
            hipLaunchKernelGGL(scan_local_kernel, dim3((unsigned)blocks), dim3(256), 0, st, counts.as<int>(), n_words,
                               counts.as<int>(), sums.as<int>());
            hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(256), 0, st, sums.as<int>(), blocks);
            hipLaunchKernelGGL(word_bases_kernel, grid_for(n_words), dim3(256), 0, st, counts.as<int>(), sums.as<int>(), n_words,
                               words.as<FeatureWord>());
        }
        const int64_t group = fill_group(M, d, nnz_c);
        for (int64_t r0 = 0; r0 < M && nnz_c > 0; r0 += group) {
            const int64_t r1 = (r0 + group < M) ? r0 + group : M;
            hipLaunchKernelGGL(centre_entries_kernel, dim3((unsigned)((r1 - r0 + 3) / 4)), dim3(256), 0, st, c_indptr, c_indices, r0, r1,
                               words.as<FeatureWord>(), number.as<int>(), row.as<int>(), place.as<int>(), col_ptr.as<int>());
        }
        hipLaunchKernelGGL(scan_local_kernel, dim3((unsigned)fill_blocks), dim3(256), 0, st, col_ptr.as<int>(), features + 1,
                           col_ptr.as<int>(), sums.as<int>());
        hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(256), 0, st, sums.as<int>(), fill_blocks);
        hipLaunchKernelGGL(scan_add_kernel, grid_for(features / 4 + 1), dim3(256), 0, st, col_ptr.as<int>(), features + 1, sums.as<int>());
        if (nnz_c > 0)
            hipLaunchKernelGGL(csc_fill_kernel, grid_for(nnz_c), dim3(256), 0, st, number.as<int>(), place.as<int>(), row.as<int>(),
                               c_values, nnz_c, col_ptr.as<int>(), csc_row.as<int>(), csc_val.as<float>());
        return hipGetLastError() == hipSuccess ? KNM_OK : fail(ctx, KNM_HIP_ERROR, "centre lists launch");
    }
};

} // namespace

// Everything the two sweeps of one (X, C, sigma) need, prepared once: validated structure, norms,
// centre lists, accumulators.
struct SparseProducts::Impl {
    knm_ctx *ctx = nullptr;
    const int64_t *x_indptr = nullptr, *x_indices = nullptr;
    const float *x_values = nullptr;
    int64_t n = 0, M = 0;
    float inv2s2 = 0.0f, inv_s2 = 0.0f;
    int64_t wgs = 0;
    CentreLists lists;
    DevBuf xn, cn, xa, cb, acc, part, tmp, work_count, work_pairs, work_q0, work_len, work_val;
    // pair lists (null: the sweeps walk the centre lists each time)
    DevBuf pair_off, pair_count, pair_part;
    int pair_ranges = 0, pair_width = 0, pair_wgs = 0; // of pair_columns_kernel
    void *pairs = nullptr;
    bool registered = false;
    ~Impl()
    {
        if (registered) spare_remove(ctx, 0, &pairs);
        if (pairs) pool_give(ctx, pairs);
    }
    // head features: dense head parts XH (n x Hn), CH (M x Hn), factors of the tail norms, per-row
    // head counts, and the vectors of the dense product (tmp_m over the centres, dense_n / tmp_n over
    // the rows)
    int Hn = 0;
    float sigma = 0.0f;
    DevBuf head_feat, head_count, XH, CH, xat, cbt, tmp_m, dense_n, dense_m, tmp_n;
    std::unique_ptr<SweepShare> share; // of the dense head product
    DevBuf col_base, col_scattered; // column sweep: all-pairs part and scattered terms, fp64 over the centres

    int rank_one_sum(const float *ev, const float *vec, int64_t ldv, int64_t rows, double *out)
    {
        double host[256];
        hipStream_t st = ctx->stream;
        hipLaunchKernelGGL(weighted_sum_kernel, dim3(256), dim3(256), 0, st, ev, vec, ldv, rows, part.as<double>());
        hipError_t err = hipMemcpyAsync(host, part.p, sizeof(double) * 256, hipMemcpyDeviceToHost, st);
        if (err == hipSuccess) err = hipStreamSynchronize(st);
        if (err != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "rank-one sum", err);
        double s = 0.0;
        for (int i = 0; i < 256; ++i) s += host[i];
        *out = s;
        return KNM_OK;
    }
    // Chooses the head features from the centre lists and builds CH.  A feature qualifies with a
    // list of at least max(16, M / 160) centres; the kMaxHead longest are taken if, on the estimate
    // that a feature is as frequent in the rows as in the centres, they would cost more pair updates
    // (n / M sum_h len_h^2) than the dense product costs entries (n M / 128 at the measured rates).
    int choose_head(int64_t nnz_c, int max_head, int *min_len_out)
    {
        hipStream_t st = ctx->stream;
        Hn = 0;
        const int min_len = (int)(M / 160 > 16 ? M / 160 : 16);
        *min_len_out = min_len;
        if (max_head <= 0 || nnz_c < min_len) return KNM_OK;
        if (max_head > kMaxHead) max_head = kMaxHead;
        const int cap = (int)(nnz_c / min_len) + 1; // no more features than this can have such lists
        DevBuf count, cand;
        if (count.alloc(ctx, sizeof(int)) != hipSuccess || cand.alloc(ctx, sizeof(int) * 3 * (size_t)cap) != hipSuccess) {
            (void)hipGetLastError();
            return fail(ctx, KNM_ALLOC, "hipMalloc(head candidates)");
        }
        hipError_t e = hipMemsetAsync(count.p, 0, sizeof(int), st);
        if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipMemsetAsync", e);
        hipLaunchKernelGGL(head_candidates_kernel, grid_for(lists.features), dim3(256), 0, st, lists.col_ptr.as<int>(),
                           lists.features, min_len, cap, count.as<int>(), cand.as<int>());
        int found = 0;
        e = hipMemcpyAsync(&found, count.p, sizeof(int), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "head candidates", e);
        if (found <= 0) return KNM_OK;
        if (found > cap) found = cap;
        std::vector<int> host(3 * (size_t)found);
        e = hipMemcpy(host.data(), cand.p, sizeof(int) * host.size(), hipMemcpyDeviceToHost);
        if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "head candidates", e);
        struct Cand { int feat, q0, len; };
        std::vector<Cand> cs((size_t)found);
        for (int i = 0; i < found; ++i) cs[i] = {host[3 * i], host[3 * i + 1], host[3 * i + 2]};
        // longest first; equal lengths by feature id, so the choice does not depend on the order
        // in which the candidates were found
        std::sort(cs.begin(), cs.end(), [](const Cand &x, const Cand &y) { return x.len != y.len ? x.len > y.len : x.feat < y.feat; });
        if ((int)cs.size() > max_head) cs.resize((size_t)max_head);
        double sq = 0.0;
        for (const Cand &c : cs) sq += (double)c.len * (double)c.len;
        if (sq * 128.0 < (double)M * (double)M) return KNM_OK;
        std::sort(cs.begin(), cs.end(), [](const Cand &x, const Cand &y) { return x.feat < y.feat; });
        Hn = (int)cs.size();
        HeadLists hl;
        int feats[kMaxHead], longest = 0;
        for (int h = 0; h < kMaxHead; ++h) {
            hl.q0[h] = h < Hn ? cs[h].q0 : 0;
            hl.len[h] = h < Hn ? cs[h].len : 0;
            feats[h] = h < Hn ? cs[h].feat : 0;
            if (hl.len[h] > longest) longest = hl.len[h];
        }
        if (head_feat.alloc(ctx, sizeof(int) * kMaxHead) != hipSuccess || CH.alloc(ctx, sizeof(float) * (size_t)M * Hn) != hipSuccess ||
            XH.alloc(ctx, sizeof(float) * (size_t)n * Hn) != hipSuccess || xat.alloc(ctx, sizeof(float) * n) != hipSuccess ||
            cbt.alloc(ctx, sizeof(float) * M) != hipSuccess || tmp_m.alloc(ctx, sizeof(float) * M) != hipSuccess ||
            dense_m.alloc(ctx, sizeof(float) * M) != hipSuccess || dense_n.alloc(ctx, sizeof(float) * n) != hipSuccess ||
            tmp_n.alloc(ctx, sizeof(float) * n) != hipSuccess) {
            (void)hipGetLastError();
            return fail(ctx, KNM_ALLOC, "hipMalloc(head features)");
        }
        e = hipMemcpy(head_feat.p, feats, sizeof(int) * kMaxHead, hipMemcpyHostToDevice);
        if (e == hipSuccess) e = hipMemsetAsync(CH.p, 0, sizeof(float) * (size_t)M * Hn, st);
        if (e == hipSuccess) e = hipMemsetAsync(XH.p, 0, sizeof(float) * (size_t)n * Hn, st);
        if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "head features", e);
        hipLaunchKernelGGL(head_centres_kernel, dim3((unsigned)((longest + 255) / 256), (unsigned)Hn), dim3(256), 0, st, hl, Hn,
                           lists.csc_row.as<int>(), lists.csc_val.as<float>(), CH.as<float>());
        return hipGetLastError() == hipSuccess ? KNM_OK : fail(ctx, KNM_HIP_ERROR, "head_centres_kernel launch");
    }
    SparseArgs args()
    {
        SparseArgs a;
        a.x_indptr = x_indptr;
        a.work_count = work_count.as<int>();
        a.work_q0 = work_q0.as<int>();
        a.work_len = work_len.as<int>();
        a.work_val = work_val.as<float>();
        a.work_pairs = work_pairs.as<int>();
        a.scattered = nullptr;
        a.Hn = Hn;
        a.head_count = head_count.as<int>();
        a.CH = CH.as<float>();
        a.tail_factor = xat.as<float>();
        a.dense = dense_n.as<float>();
        a.n = n;
        a.M = M;
        a.csc_row = lists.csc_row.as<int>();
        a.csc_val = lists.csc_val.as<float>();
        a.xn = xn.as<float>();
        a.cn = cn.as<float>();
        a.xa = xa.as<float>();
        a.acc = acc.as<float>();
        a.inv2s2 = inv2s2;
        a.inv_s2 = inv_s2;
        a.pair_off = pair_off.as<int>();
        a.pair_count = pair_count.as<int>();
        a.pairs = static_cast<SparsePair *>(pairs);
        return a;
    }
    // Writes the pairs down, if there is room for them (`total`: no more than this).
    int form_pairs(unsigned long long total)
    {
        hipStream_t st = ctx->stream;
        if (total == 0 || total > kMaxPairs || M > 16 * kPairWidth) return KNM_OK;
        const int64_t blocks = (n + kScanChunk - 1) / kScanChunk;
        pair_ranges = (int)((M + kPairWidth - 1) / kPairWidth);
        pair_width = (int)((M + pair_ranges - 1) / pair_ranges);
        // one workgroup per CU, two where their LDS lets them, over all ranges; no more than have rows
        pair_wgs = (pair_width > kPairWidth / 2 ? 256 : 512) / pair_ranges;
        if (pair_wgs < 16) pair_wgs = 16;
        if (pair_wgs > (n + 63) / 64) pair_wgs = (int)((n + 63) / 64);
        DevBuf sums;
        void *p = nullptr;
        if (sums.alloc(ctx, sizeof(int) * (size_t)blocks) != hipSuccess ||
            pair_count.alloc(ctx, sizeof(int) * (size_t)n) != hipSuccess ||
            pair_part.alloc(ctx, sizeof(double) * (size_t)pair_wgs * (size_t)M) != hipSuccess ||
            pool_take(ctx, sizeof(SparsePair) * (size_t)total, &p, PoolUse::kForSpeed) != hipSuccess) {
            (void)hipGetLastError();
            return KNM_OK; // no room: every sweep walks
        }
        pairs = p;
        registered = spare_add(ctx, 0, &pairs); // given up when something else finds no room
        int *off = pair_off.as<int>();
        hipLaunchKernelGGL(scan_local_kernel, dim3((unsigned)blocks), dim3(256), 0, st, off, n, off, sums.as<int>());
        hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(256), 0, st, sums.as<int>(), blocks);
        hipLaunchKernelGGL(scan_add_kernel, grid_for((n + 3) / 4), dim3(256), 0, st, off, n, sums.as<int>());
        hipLaunchKernelGGL(sparse_sweep_kernel<kFormPairs>, dim3((unsigned)wgs), dim3(kSpThreads), 0, st, args());
        return hipGetLastError() == hipSuccess ? KNM_OK : fail(ctx, KNM_HIP_ERROR, "pair lists launch");
    }
};

SparseProducts::SparseProducts() : impl(new Impl()) {}
SparseProducts::~SparseProducts() { delete impl; }

int SparseProducts::prepare(knm_ctx *ctx, const int64_t *x_indptr, const int64_t *x_indices, const float *x_values,
                            int64_t n, const int64_t *c_indptr, const int64_t *c_indices, const float *c_values,
                            int64_t M, int64_t d, float sigma, int uses)
{
    // the closed form of the rank-one part belongs to the Gaussian kernel
    if (ctx->kernel_kind != KNM_KERNEL_GAUSSIAN)
        return fail(ctx, KNM_UNSUPPORTED, "sparse inputs: Gaussian kernel only");
    Impl &s = *impl;
    s.ctx = ctx;
    s.x_indptr = x_indptr;
    s.x_indices = x_indices;
    s.x_values = x_values;
    s.n = n;
    s.M = M;
    s.inv2s2 = 1.0f / (2.0f * sigma * sigma);
    s.inv_s2 = 1.0f / (sigma * sigma);
    hipStream_t st = ctx->stream;
    int64_t nnz_x = 0, nnz_c = 0;
    int stat = check_csr(ctx, x_indptr, x_indices, n, d, &nnz_x);
    if (!stat) stat = check_csr(ctx, c_indptr, c_indices, M, d, &nnz_c);
    if (stat) return stat;
    // grid: enough wavefronts to fill the chip, each with a private accumulator over the centres
    s.wgs = (n + kSpWaves - 1) / kSpWaves;
    if (s.wgs > 2048) s.wgs = 2048; // 8 workgroups per CU: the sweep is bound by memory latency
    const int64_t waves = s.wgs * kSpWaves;
    if (s.xn.alloc(ctx, sizeof(float) * n) != hipSuccess || s.cn.alloc(ctx, sizeof(float) * M) != hipSuccess ||
        s.xa.alloc(ctx, sizeof(float) * n) != hipSuccess || s.cb.alloc(ctx, sizeof(float) * M) != hipSuccess ||
        s.acc.alloc(ctx, sizeof(float) * waves * M) != hipSuccess || s.part.alloc(ctx, sizeof(double) * 256) != hipSuccess ||
        s.tmp.alloc(ctx, sizeof(float) * n) != hipSuccess || s.col_base.alloc(ctx, sizeof(double) * M) != hipSuccess ||
        s.col_scattered.alloc(ctx, sizeof(double) * M) != hipSuccess) {
        (void)hipGetLastError();
        return fail(ctx, KNM_ALLOC, "hipMalloc(sparse workspace)");
    }
    hipLaunchKernelGGL(row_norms_kernel, row_pass_grid(n), dim3(256), 0, st, x_indptr, x_values, n, s.xn.as<float>());
    hipLaunchKernelGGL(row_norms_kernel, row_pass_grid(M), dim3(256), 0, st, c_indptr, c_values, M, s.cn.as<float>());
    hipLaunchKernelGGL(norm_factor_kernel, grid_for(n), dim3(256), 0, st, s.xn.as<float>(), n, s.inv2s2, s.xa.as<float>());
    hipLaunchKernelGGL(norm_factor_kernel, grid_for(M), dim3(256), 0, st, s.cn.as<float>(), M, s.inv2s2, s.cb.as<float>());
    stat = s.lists.build(ctx, c_indptr, c_indices, c_values, M, d, nnz_c);
    if (stat) return stat;
    s.sigma = sigma;
    int head_min_len = 0;
    stat = s.choose_head(nnz_c, ctx->sparse_head_max, &head_min_len);
    if (stat) return stat;
    const size_t work = (size_t)(nnz_x > 0 ? nnz_x : 1);
    if (s.work_count.alloc(ctx, sizeof(int) * n) != hipSuccess || s.head_count.alloc(ctx, sizeof(int) * n) != hipSuccess ||
        s.work_pairs.alloc(ctx, sizeof(int) * n) != hipSuccess ||
        s.pair_off.alloc(ctx, sizeof(int) * n) != hipSuccess || s.work_q0.alloc(ctx, sizeof(int) * work) != hipSuccess || s.work_len.alloc(ctx, sizeof(int) * work) != hipSuccess ||
        s.work_val.alloc(ctx, sizeof(float) * work) != hipSuccess) {
        (void)hipGetLastError();
        return fail(ctx, KNM_ALLOC, "hipMalloc(sparse work list)");
    }
    // in the partial sums' room: largest head norm term, and from the next cache line on the number of pairs
    unsigned long long words[(1 + kTotals) * kTotalStride] = {};
    static_assert(sizeof(words) <= sizeof(double) * 256, "room of the partial sums");
    unsigned *const worst_dev = s.part.as<unsigned>();
    unsigned long long *const totals_dev = uses > 1 ? s.part.as<unsigned long long>() + kTotalStride : nullptr;
    auto read_words = [&]() -> int {
        hipError_t e = hipMemcpyAsync(words, s.part.p, sizeof(words), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        return e == hipSuccess ? KNM_OK : fail(ctx, KNM_HIP_ERROR, "sparse work list", e);
    };
    auto build_work = [&]() {
        if (hipMemsetAsync(s.part.p, 0, sizeof(words), st) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipMemsetAsync");
        hipLaunchKernelGGL(build_work_kernel, dim3((unsigned)s.wgs), dim3(kSpThreads), 0, st, x_indptr, x_indices, x_values, n,
                           s.lists.words.as<FeatureWord>(), s.lists.col_ptr.as<int>(), s.head_feat.as<int>(), s.Hn, head_min_len, s.work_count.as<int>(),
                           s.work_pairs.as<int>(), s.head_count.as<int>(), s.work_q0.as<int>(), s.work_len.as<int>(),
                           s.work_val.as<float>(), s.XH.as<float>(), M, s.pair_off.as<int>(), totals_dev);
        return hipGetLastError() == hipSuccess ? KNM_OK : fail(ctx, KNM_HIP_ERROR, "work list launch");
    };
    stat = build_work();
    if (stat) return stat;
    if (s.Hn > 0) {
        // The dense product forms its exponent from the norm expansion, whose rounding error grows
        // with the head parts' norm terms |x^H|^2 / 2 sigma^2 (about 1e-7 of them): beyond 50 the
        // head features go back into the sparse walk, which has no such cancellation.
        hipLaunchKernelGGL(tail_factor_kernel, grid_for(n), dim3(256), 0, st, s.xn.as<float>(), s.XH.as<float>(), s.Hn, n,
                           s.inv2s2, s.xat.as<float>(), worst_dev);
        hipLaunchKernelGGL(tail_factor_kernel, grid_for(M), dim3(256), 0, st, s.cn.as<float>(), s.CH.as<float>(), s.Hn, M,
                           s.inv2s2, s.cbt.as<float>(), worst_dev);
        stat = read_words();
        if (stat) return stat;
        const unsigned worst_bits = (unsigned)words[0];
        float worst = 0.0f;
        memcpy(&worst, &worst_bits, sizeof(float));
        if (!(worst <= 50.0f)) {
            s.Hn = 0;
            stat = build_work();
            if (!stat && uses > 1) stat = read_words();
            if (stat) return stat;
        }
    } else if (uses > 1) {
        stat = read_words();
        if (stat) return stat;
    }
    if (s.Hn > 0)
        s.share.reset(new (std::nothrow) SweepShare(ctx, s.XH.as<float>(), n, s.Hn, s.CH.as<float>(), M, s.Hn, s.Hn, sigma, 1, true));
    if (s.Hn > 0 && !s.share) return fail(ctx, KNM_ALLOC, "host allocation");
    unsigned long long total = 0;
    for (int k = 1; k <= kTotals; ++k) total += words[k * kTotalStride];
    return uses > 1 ? s.form_pairs(total) : KNM_OK;
}

// W (n x t, row-major) = K V
int SparseProducts::v(const float *V, int t, float *W)
{
    Impl &s = *impl;
    for (int c = 0; c < t; ++c) {
        double sum = 0.0;
        if (s.Hn > 0) {
            // all pairs: a^T_i sum_j k(x^H_i, c^H_j) b^T_j v_j on the dense engine
            hipLaunchKernelGGL(scale_kernel, grid_for(s.M), dim3(256), 0, s.ctx->stream, s.cbt.as<float>(), V + c, (int64_t)t,
                               s.M, s.tmp_m.as<float>(), (int64_t)1);
            const ShareScope scope(*s.share);
            int stat = do_knm_v(s.ctx, s.XH.as<float>(), s.n, s.Hn, s.Hn, s.CH.as<float>(), s.M, s.Hn, s.sigma,
                                s.tmp_m.as<float>(), 1, s.dense_n.as<float>());
            if (stat) return stat;
        } else {
            int stat = s.rank_one_sum(s.cb.as<float>(), V + c, t, s.M, &sum);
            if (stat) return stat;
        }
        SparseArgs a = s.args();
        a.vec = V + c;
        a.ldv = t;
        a.out = W + c;
        a.ldo = t;
        a.s_rank_one = sum;
        if (s.pairs) hipLaunchKernelGGL(pair_rows_kernel, row_pass_grid(s.n), dim3(256), 0, s.ctx->stream, a);
        else hipLaunchKernelGGL(sparse_sweep_kernel<kRowSweep>, dim3((unsigned)s.wgs), dim3(kSpThreads), 0, s.ctx->stream, a);
    }
    return hipGetLastError() == hipSuccess ? KNM_OK : fail(s.ctx, KNM_HIP_ERROR, "sparse row sweep launch");
}

// U (M x t, row-major) = K^T (wgt .* W), wgt over the rows of X or null
int SparseProducts::t_w(const float *W, const float *wgt, int t, float *U)
{
    Impl &s = *impl;
    hipStream_t st = s.ctx->stream;
    for (int c = 0; c < t; ++c) {
        const float *w = W + c;
        int64_t ldw = t;
        if (wgt) {
            hipLaunchKernelGGL(weigh_kernel, grid_for(s.n), dim3(256), 0, st, W + c, (int64_t)t, wgt, s.n, s.tmp.as<float>());
            w = s.tmp.as<float>();
            ldw = 1;
        }
        if (s.Hn > 0) {
            // all pairs: b^T_j sum_i k(x^H_i, c^H_j) a^T_i w_i on the dense engine
            hipLaunchKernelGGL(scale_kernel, grid_for(s.n), dim3(256), 0, st, s.xat.as<float>(), w, ldw, s.n,
                               s.tmp_n.as<float>(), (int64_t)1);
            const ShareScope scope(*s.share);
            int stat = do_knm_t_w(s.ctx, s.XH.as<float>(), s.n, s.Hn, s.Hn, s.CH.as<float>(), s.M, s.Hn, s.sigma,
                                  s.tmp_n.as<float>(), nullptr, 1, s.dense_m.as<float>());
            if (stat) return stat;
            hipLaunchKernelGGL(column_base_kernel, grid_for(s.M), dim3(256), 0, st, s.cbt.as<float>(), s.dense_m.as<float>(), 0.0,
                               s.M, s.col_base.as<double>());
        } else {
            double sum = 0.0;
            int stat = s.rank_one_sum(s.xa.as<float>(), w, ldw, s.n, &sum);
            if (stat) return stat;
            hipLaunchKernelGGL(column_base_kernel, grid_for(s.M), dim3(256), 0, st, s.cb.as<float>(), (const float *)nullptr, sum,
                               s.M, s.col_base.as<double>());
        }
        hipError_t e = s.pairs ? hipSuccess : hipMemsetAsync(s.col_scattered.p, 0, sizeof(double) * s.M, st);
        if (e != hipSuccess) return fail(s.ctx, KNM_HIP_ERROR, "hipMemsetAsync", e);
        SparseArgs a = s.args();
        a.vec = w;
        a.ldv = ldw;
        a.out = nullptr;
        a.ldo = 0;
        a.scattered = s.col_scattered.as<double>();
        a.s_rank_one = 0.0;
        if (s.pairs) {
            const size_t lds = sizeof(double) * (size_t)s.pair_width;
            e = hipFuncSetAttribute(reinterpret_cast<const void *>(pair_columns_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kPairWidth * (int)sizeof(double));
            if (e != hipSuccess) return fail(s.ctx, KNM_HIP_ERROR, "hipFuncSetAttribute", e);
            hipLaunchKernelGGL(pair_columns_kernel, dim3((unsigned)s.pair_wgs, (unsigned)s.pair_ranges), dim3(kPairThreads), lds, st, a, s.pair_width,
                               s.pair_part.as<double>());
            e = launch_merge(nullptr, s.pair_part.as<double>(), s.pair_wgs, s.M, 1, nullptr, s.col_scattered.as<double>(), 1, s.M, st);
            if (e != hipSuccess) return fail(s.ctx, KNM_HIP_ERROR, "launch_merge", e);
        } else hipLaunchKernelGGL(sparse_sweep_kernel<kColumnSweep>, dim3((unsigned)s.wgs), dim3(kSpThreads), 0, st, a);
        hipLaunchKernelGGL(column_finish_kernel, grid_for(s.M), dim3(256), 0, st, s.col_base.as<double>(),
                           s.col_scattered.as<double>(), s.M, U + c, (int64_t)t);
    }
    return hipGetLastError() == hipSuccess ? KNM_OK : fail(s.ctx, KNM_HIP_ERROR, "sparse column sweep launch");
}

// Upper triangle of K (M x M, column-major with leading dimension ldk, fp64) = k(C, C) + jitter I for CSR centres
int sparse_kmm(knm_ctx *ctx, const int64_t *c_indptr, const int64_t *c_indices, const float *c_values, int64_t M,
               int64_t d, float sigma, double jitter, double *K, int64_t ldk)
{
    if (ctx->kernel_kind != KNM_KERNEL_GAUSSIAN)
        return fail(ctx, KNM_UNSUPPORTED, "sparse inputs: Gaussian kernel only");
    hipStream_t st = ctx->stream;
    int64_t nnz_c = 0;
    int stat = check_csr(ctx, c_indptr, c_indices, M, d, &nnz_c);
    if (stat) return stat;
    CentreLists lists;
    stat = lists.build(ctx, c_indptr, c_indices, c_values, M, d, nnz_c);
    if (stat) return stat;
    int64_t wgs = (M + kSpWaves - 1) / kSpWaves;
    if (wgs > 1024) wgs = 1024;
    const int64_t waves = wgs * kSpWaves;
    DevBuf cn, acc;
    if (cn.alloc(ctx, sizeof(double) * M) != hipSuccess || acc.alloc(ctx, sizeof(double) * waves * M) != hipSuccess) {
        (void)hipGetLastError();
        return fail(ctx, KNM_ALLOC, "hipMalloc(sparse K_MM workspace)");
    }
    hipLaunchKernelGGL(row_norms_f64_kernel, grid_for(M), dim3(256), 0, st, c_indptr, c_values, M, cn.as<double>());
    hipError_t e = hipMemsetAsync(acc.p, 0, sizeof(double) * waves * M, st);
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipMemsetAsync", e);
    hipLaunchKernelGGL(sparse_kmm_kernel, dim3((unsigned)wgs), dim3(kSpThreads), 0, st, c_indptr, lists.number.as<int>(), c_values, M,
                       lists.col_ptr.as<int>(), lists.csc_row.as<int>(), lists.csc_val.as<float>(), cn.as<double>(),
                       1.0 / (2.0 * (double)sigma * (double)sigma), jitter, acc.as<double>(), K, ldk);
    e = hipGetLastError();
    return e == hipSuccess ? KNM_OK : fail(ctx, KNM_HIP_ERROR, "sparse K_MM", e);
}

} // namespace knm

extern "C" int knm_prod_csr(knm_ctx *ctx, const int64_t *x_indptr, const int64_t *x_indices, const float *x_values,
                            int64_t n, const int64_t *c_indptr, const int64_t *c_indices, const float *c_values,
                            int64_t M, int64_t d, float sigma, const float *V, int t, float *W_or_null, float *U)
{
    using namespace knm;
    if (!ctx) return KNM_INVALID_ARG;
    if (!x_indptr || !c_indptr || !V || !U || n <= 0 || M <= 0 || d <= 0 || t <= 0 || !(sigma > 0.0f))
        return fail(ctx, KNM_INVALID_ARG, "bad shape or pointer");
    if (d >= 0x7fffffffLL || M >= 0x7fffffffLL) return fail(ctx, KNM_UNSUPPORTED, "d or M beyond 2^31 - 2");
    if (t > knm_max_t()) return fail(ctx, KNM_UNSUPPORTED, "t above compiled maximum");
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipSetDevice");
    SparseProducts ops;
    int st = ops.prepare(ctx, x_indptr, x_indices, x_values, n, c_indptr, c_indices, c_values, M, d, sigma, 2);
    if (st) return st;
    float *W = W_or_null;
    if (!W) {
        st = ensure(ctx, &ctx->w_buf, &ctx->w_bytes, sizeof(float) * (size_t)n * t);
        if (st) return st;
        W = ctx->w_buf;
    }
    st = ops.v(V, t, W);
    if (!st) st = ops.t_w(W, nullptr, t, U);
    if (st) return st;
    hipError_t e = hipStreamSynchronize(ctx->stream);
    if (e == hipSuccess) e = hipGetLastError();
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "sparse product", e);
    return KNM_OK;
}
