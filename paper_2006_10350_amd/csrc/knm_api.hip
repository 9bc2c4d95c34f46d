// C ABI of libknm: context, workspace and the kernel-matrix-vector products.
#include <dlfcn.h>

#include <chrono>
#include <cmath>
#include <cstddef>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <utility>

#include "knm_internal.h"

namespace knm {

namespace {
struct MarkerApi {
    int (*push)(const char *) = nullptr;
    int (*pop)() = nullptr;
};
const MarkerApi &marker_api()
{
    static MarkerApi api;
    static std::once_flag once;
    std::call_once(once, [] {
        const char *want = std::getenv("KNM_MARKERS");
        if (!want || !*want || std::strcmp(want, "0") == 0) return;
        for (const char *lib : {"librocprofiler-sdk-roctx.so", "libroctx64.so"}) {
            void *h = dlopen(lib, RTLD_NOW | RTLD_GLOBAL);
            if (!h) continue;
            auto push = reinterpret_cast<int (*)(const char *)>(dlsym(h, "roctxRangePushA"));
            auto pop = reinterpret_cast<int (*)()>(dlsym(h, "roctxRangePop"));
            if (push && pop) {
                api.push = push;
                api.pop = pop;
                return;
            }
        }
    });
    return api;
}
} // namespace

TraceRange::TraceRange(const char *name) : open(false)
{
    const MarkerApi &api = marker_api();
    if (api.push) {
        (void)api.push(name);
        open = true;
    }
}
TraceRange::~TraceRange()
{
    if (open) (void)marker_api().pop();
}

int fail(knm_ctx *ctx, int status, const char *what, hipError_t e)
{
    if (ctx) {
        ctx->last_error = what ? what : "";
        if (e != hipSuccess) {
            ctx->last_error += ": ";
            ctx->last_error += hipGetErrorString(e);
        }
    }
    return status;
}

// frees the idle blocks of the pool (its lock is held; hipFree waits for the device)
static void free_idle_locked(knm_ctx *ctx)
{
    for (size_t i = 0; i < ctx->pool.size();) {
        if (ctx->pool[i].used) {
            ++i;
            continue;
        }
        (void)hipFree(ctx->pool[i].p);
        ctx->pool.erase(ctx->pool.begin() + (std::ptrdiff_t)i);
    }
    ctx->pool_idle = 0;
}

// marks a block of the pool as idle (the pool's lock is held)
static void idle_locked(knm_ctx *ctx, void *p)
{
    for (auto &b : ctx->pool)
        if (b.p == p && b.used) {
            b.used = false;
            ctx->pool_idle += b.bytes;
        }
}

bool spare_add(knm_ctx *ctx, int phase, void **p)
{
    const std::lock_guard<std::mutex> lock(ctx->pool_lock);
    try {
        ctx->spare[phase].push_back(p);
    } catch (const std::bad_alloc &) {
        return false;
    }
    return true;
}
void spare_remove(knm_ctx *ctx, int phase, void **p)
{
    const std::lock_guard<std::mutex> lock(ctx->pool_lock);
    auto &list = ctx->spare[phase];
    for (size_t i = 0; i < list.size(); ++i)
        if (list[i] == p) {
            list.erase(list.begin() + (std::ptrdiff_t)i);
            return;
        }
}

// hipMalloc that gives up the idle blocks of the pool when there is no room, and then (unless optional) what the calls under way keep
// but can do without: kernel values and pair lists (formed again by every sweep from there on), then images (packed slab by
// slab from there on).  The pool's lock is held.
static hipError_t alloc_locked(knm_ctx *ctx, size_t bytes, void **out, bool optional)
{
    *out = nullptr;
    hipError_t e = hipMalloc(out, bytes);
    for (int phase = -1; e != hipSuccess && phase < (optional ? 0 : 2); ++phase) {
        (void)hipGetLastError();
        if (phase >= 0)
            for (void **p : ctx->spare[phase])
                if (*p) {
                    idle_locked(ctx, *p);
                    *p = nullptr;
                }
        if (ctx->pool_idle == 0) continue;
        free_idle_locked(ctx);
        e = hipMalloc(out, bytes);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        *out = nullptr;
    }
    return e;
}

hipError_t device_alloc(knm_ctx *ctx, size_t bytes, void **out)
{
    const std::lock_guard<std::mutex> lock(ctx->pool_lock);
    return alloc_locked(ctx, bytes, out, false);
}

int ensure(knm_ctx *ctx, float **buf, size_t *cur, size_t need)
{
    if (*cur >= need) return KNM_OK;
    if (*buf) {
        hipError_t e = hipFree(*buf);
        *buf = nullptr;
        *cur = 0;
        if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipFree(workspace)", e);
    }
    void *p = nullptr;
    hipError_t e = device_alloc(ctx, need, &p);
    if (e != hipSuccess) {
        return fail(ctx, KNM_ALLOC, "hipMalloc(workspace)", e);
    }
    *buf = static_cast<float *>(p);
    *cur = need;
    return KNM_OK;
}

static bool is_capturing(knm_ctx *ctx)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    const hipError_t e = hipStreamIsCapturing(ctx->stream, &status);
    if (e != hipSuccess) (void)hipGetLastError(); // (the null stream beside one that is captured)
    return e != hipSuccess || status != hipStreamCaptureStatusNone;
}

static size_t pool_bytes(knm_ctx *ctx, const void *p)
{
    const std::lock_guard<std::mutex> lock(ctx->pool_lock);
    for (const auto &b : ctx->pool)
        if (b.p == p) return b.bytes;
    return 0;
}

// Idle blocks beyond this are freed (30 ms per GiB once a process has gone through the card's memory: what a fit keeps has to fit), and
// beyond the second number where the card is nearly full
constexpr size_t kPoolIdleBytes = (size_t)16 << 30, kPoolIdleFull = (size_t)4 << 30;

// Whether a sixteenth of the card (18 GB) is left beside `bytes` more: kernel values, pair lists and slabs are for speed alone and leave that to
// the rest of the program, whose own allocator sees none of the idle blocks.
static bool leaves_room(size_t bytes)
{
    size_t free = 0, total = 0;
    if (hipMemGetInfo(&free, &total) == hipSuccess) return free >= bytes && free - bytes >= total / 16;
    (void)hipGetLastError();
    return false;
}

// ensure() for what is for speed alone: false, with everything as it was, where the card has no room to spare or the stream is being captured
static bool ensure_for_speed(knm_ctx *ctx, float **buf, size_t *cur, size_t need)
{
    if (*cur >= need) return true;
    if (is_capturing(ctx) || !leaves_room(need)) return false;
    void *p = nullptr;
    {
        const std::lock_guard<std::mutex> lock(ctx->pool_lock);
        if (alloc_locked(ctx, need, &p, true) != hipSuccess) return false;
    }
    if (*buf) (void)hipFree(*buf);
    *buf = static_cast<float *>(p);
    *cur = need;
    return true;
}

hipError_t pool_take(knm_ctx *ctx, size_t bytes, void **out, PoolUse use)
{
    *out = nullptr;
    bytes = (bytes + 255) & ~(size_t)255;
    if (bytes == 0) bytes = 256;
    const std::lock_guard<std::mutex> lock(ctx->pool_lock);
    // the smallest idle block that fits without wasting more than it gives
    knm_ctx::PoolBlock *best = nullptr;
    for (auto &b : ctx->pool)
        if (!b.used && b.bytes >= bytes && b.bytes <= 2 * bytes + 65536 && (best == nullptr || b.bytes < best->bytes)) best = &b;
    if (best != nullptr) {
        best->used = true;
        ctx->pool_idle -= best->bytes;
        *out = best->p;
        return hipSuccess;
    }
    if (use == PoolUse::kForSpeed && !leaves_room(bytes)) return hipErrorOutOfMemory;
    void *p = nullptr;
    const hipError_t e = alloc_locked(ctx, bytes, &p, use != PoolUse::kNeeded);
    if (e != hipSuccess) return e;
    try {
        ctx->pool.push_back({p, bytes, true});
    } catch (const std::bad_alloc &) { // the entry points are C: nothing may be thrown through them
        (void)hipFree(p);
        return hipErrorOutOfMemory;
    }
    *out = p;
    return hipSuccess;
}

void pool_give(knm_ctx *ctx, void *p)
{
    const std::lock_guard<std::mutex> lock(ctx->pool_lock);
    for (size_t i = 0; i < ctx->pool.size(); ++i) {
        auto &b = ctx->pool[i];
        if (b.p != p) continue;
        b.used = false;
        ctx->pool_idle += b.bytes;
        break;
    }
    // (how full the card is is asked at most every 50 ms: a call gives some 25 blocks back, and the answer takes 5 to 50 us)
    auto full = [&] {
        const auto now = std::chrono::steady_clock::now();
        if (now - ctx->room_asked > std::chrono::milliseconds(50)) {
            ctx->room_asked = now;
            ctx->room_left = leaves_room(0);
        }
        return !ctx->room_left;
    };
    // oldest idle blocks first (hipFree waits for the device, so nothing queued still uses them)
    auto too_many = [&] { return ctx->pool_idle > kPoolIdleBytes || (ctx->pool_idle > kPoolIdleFull && full()); };
    for (size_t i = 0; i < ctx->pool.size();) {
        if (ctx->pool[i].used) {
            ++i;
            continue;
        }
        if (!too_many()) break;
        ctx->pool_idle -= ctx->pool[i].bytes;
        (void)hipFree(ctx->pool[i].p);
        ctx->pool.erase(ctx->pool.begin() + (std::ptrdiff_t)i);
    }
}

size_t pool_idle_bytes(knm_ctx *ctx)
{
    const std::lock_guard<std::mutex> lock(ctx->pool_lock);
    return ctx->pool_idle;
}

void pool_trim(knm_ctx *ctx, size_t idle)
{
    const std::lock_guard<std::mutex> lock(ctx->pool_lock);
    for (size_t i = ctx->pool.size(); i-- > 0 && ctx->pool_idle > idle;)
        if (!ctx->pool[i].used) {
            ctx->pool_idle -= ctx->pool[i].bytes;
            (void)hipFree(ctx->pool[i].p);
            ctx->pool.erase(ctx->pool.begin() + (std::ptrdiff_t)i);
        }
}

void pool_drop(knm_ctx *ctx, void *p)
{
    const std::lock_guard<std::mutex> lock(ctx->pool_lock);
    for (size_t i = 0; i < ctx->pool.size(); ++i)
        if (ctx->pool[i].p == p) {
            (void)hipFree(p);
            ctx->pool.erase(ctx->pool.begin() + (std::ptrdiff_t)i);
            return;
        }
}

// Workspace for callers that cannot allocate (code under HIP graph capture, serving loops,
// harnesses that forbid hipMalloc): one array per GPU, held from the loading of the library to the
// end of the process.  Host code never uses this name as an address: knm_create looks up the
// device's own copy with hipGetSymbolAddress and keeps the pointer in the context.
constexpr size_t kStaticScratchBytes = (size_t)64 << 20;
constexpr size_t kVectorImageCap = (size_t)16 << 30; // largest packed vector image the library allocates
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// One piece of a sweep's workspace: grown on demand in the context's own buffer, or, in a call that
// must not allocate, carved from the static scratch (KNM_UNSUPPORTED if it does not fit).
static int acquire(knm_ctx *ctx, float **buf, size_t *cur, size_t need, float **out)
{
    if (!ctx->static_mode) {
        int st = ensure(ctx, buf, cur, need);
        *out = *buf;
        return st;
    }
    const size_t at = (ctx->static_used + 255) & ~(size_t)255;
    if (ctx->static_ws == nullptr || at + need > kStaticScratchBytes)
        return fail(ctx, KNM_UNSUPPORTED, "problem too large for the static scratch of the allocation-free entry point");
    *out = reinterpret_cast<float *>(ctx->static_ws + at);
    ctx->static_used = at + need;
    return KNM_OK;
}

// K-loop engine for several columns or for d beyond what the register-resident engine of the
// selected arithmetic holds (44 features for the split-fp16 one, 64 for fp32)
bool use_gemm_engine(int d, int t, int cross_term, int kind)
{
    // (the kernels of r = |x - c| run on the register-resident engine only with the split-fp16 cross
    // term, and up to the d its two smaller layouts hold without register spills)
    if (kind != KNM_KERNEL_GAUSSIAN && (cross_term != KNM_CROSS_F16X3 || d > f16_radial_max_d())) return true;
    return t > 1 || d > (cross_term == KNM_CROSS_F16X3 ? f16_max_d() : small_max_d());
}

// Sweeps whose operands are packed into images first, and the bytes of a point there: the split-fp16 engines, and in the fp32 mode the
// register-resident engine that has fp32 numbers in three bf16 parts, where it gains more than that costs.
static bool packs_images(int64_t nF, int64_t nS, int d, int t, int cross_term, int kind)
{
    if (cross_term == KNM_CROSS_F16X3) return true;
    return !use_gemm_engine(d, t, cross_term, kind) && b16_pays((double)nF * (double)nS, d);
}
static size_t image_bytes_per_point(int d, int t, int cross_term, int kind)
{
    if (cross_term != KNM_CROSS_F16X3) return b16_pack_bytes_per_point(d);
    return use_gemm_engine(d, t, cross_term, kind) ? gemm_f16_pack_bytes_per_point(d) : f16_pack_bytes_per_point(d);
}

// Chunking of the stream dimension.  More chunks = more workgroups and shorter fp32 running sums; each chunk costs one partial
// vector that the merge pass adds up in fp64.
struct ChunkGrid {
    int64_t stage, per_block, blocks, stages; // points per stage and per fixed block, fixed blocks, stages in all
    int64_t min_chunks;
};
static ChunkGrid chunk_grid(int64_t nF, int64_t nS, int d, int t, int cross_term, int kind)
{
    ChunkGrid g;
    const bool gemm = use_gemm_engine(d, t, cross_term, kind);
    g.stage = gemm ? gemm_stage_points() : (cross_term == KNM_CROSS_F16X3 ? f16_stage_points(d, kind) : stage_points());
    g.per_block = gemm ? gemm_fixed_per_block() : fixed_per_block(d);
    g.blocks = (nF + g.per_block - 1) / g.per_block;
    g.stages = (nS + g.stage - 1) / g.stage;
    const int64_t max_len = (int64_t)1 << 18; // bound the length of a per-lane fp32 running sum
    g.min_chunks = (nS + max_len - 1) / max_len;
    return g;
}

// Chunks of at least 2048 points, 4096 workgroups where the stream is long enough: fewer partials than choose_chunks, for
// calls whose workspace is limited.
static int64_t choose_chunks_compact(int64_t nF, int64_t nS, int d, int t, int cross_term, int kind, int64_t *chunk_len)
{
    const bool gemm = use_gemm_engine(d, t, cross_term, kind);
    const ChunkGrid g = chunk_grid(nF, nS, d, t, cross_term, kind);
    const int64_t min_len = gemm ? 16 * g.stage : 2048;
    int64_t chunks = (4096 + g.blocks - 1) / g.blocks;
    if (gemm && chunks < 16) chunks = 16;
    const int64_t max_chunks_by_len = (nS + min_len - 1) / min_len;
    if (chunks > max_chunks_by_len) chunks = max_chunks_by_len;
    if (chunks < g.min_chunks) chunks = g.min_chunks;
    int64_t len = (nS + chunks - 1) / chunks;
    len = (len + g.stage - 1) / g.stage * g.stage;
    *chunk_len = len;
    return (nS + len - 1) / len;
}

// The number of chunks is the one with the least estimated time among those that make about 1, 2, ... 16 rounds of the workgroups
// the chip holds at once, the smallest numbers and multiples of 8.  The estimate: rounds x stages x time of a stage, where a last round that
// takes at most half of the places counts half because its workgroups have a CU to themselves, and part of a round more because
// workgroups do not end together (measured: 79 blocks, 2.0 rounds 3.75 ms, 4.0 3.47, 4.9 3.27, 6.0 3.37, 6.9 3.27); the start
// and end of a workgroup; partials written and merged; and for the K-loop engine what the sharing of operands in an XCD's L2 loses
// (see PatchMap) with fewer than 8 chunks (d = 784: 4 chunks 32 % slower), in a last group of fewer than 8 (18 %), and in
// long chunks, along which workgroups drift apart (2 % per doubling), all in proportion to d.  Against the best of 1 to 128 chunks
// at d = 50, 100, 200, 440 and 784, 1 and 10 columns, 60k x 10k, 300k x 3k and 15k x 15k points, both sweeps: within 2 % in 59 of
// 60, 4.7 % in one.  n = 60k, d = 784, M = 10k, 10 columns ran
// 1175 workgroups of 16 tiles on 512 places: 2.48 ms per sweep, 2.0 ms cut finer.
// (any_length: the choice by time alone, whatever the length of fp32 sums; parts: of the engine that has fp32 numbers in three parts)
static int64_t choose_chunks_by_time(int64_t nF, int64_t nS, int d, int t, int cross_term, int kind, bool any_length, bool parts, int64_t *chunk_len)
{
    const bool gemm = use_gemm_engine(d, t, cross_term, kind);
    const bool f16 = cross_term == KNM_CROSS_F16X3;
    const ChunkGrid g = chunk_grid(nF, nS, d, t, cross_term, kind);
    // workgroups per CU and microseconds of a stage (K-loop engines: of a tile) of one of them on a full chip, from the rates of
    // the engines (ps per kernel entry) on large problems
    int per_cu = 2;
    double stage_us, wg_us = 5.0, uneven = 0.2;
    if (gemm) {
        const double kc = (double)((d + 15) / 16);
        const int tl = f16 && t > gemm_f16_max_t(kind) ? gemm_f16_max_t(kind) : (!f16 && t > gemm_max_t() ? gemm_max_t() : t);
        double cycles; // per tile and SIMD
        if (f16) {
            per_cu = gemm_f16_workgroups_per_cu(d, tl, kind);
            const bool mc = gemm_f16_matrix_reduction(d, tl);
            cycles = 256.0 + 900.0 * kc + (mc ? 3600.0 + 48.0 * 32.0 * ((tl + 31) / 32) : 128.0 * (14.0 + 4.0 * tl));
        } else {
            cycles = 4200.0 * kc + 128.0 * (14.0 + 4.0 * tl);
        }
        if (kind != KNM_KERNEL_GAUSSIAN) cycles += 128.0 * 16.0;
        stage_us = per_cu * cycles / 2100.0;
        wg_us = per_cu > 1 ? 6.0 : 8.0;
        uneven = 0.4;
    } else {
        if (f16) per_cu = f16_workgroups_per_cu(d, kind);
        if (parts) per_cu = b16_workgroups_per_cu(d);
        const double ps = (f16 ? (d <= 12 ? 0.106 : d <= 28 ? 0.167 : 0.22) : parts ? 0.085 + 0.0075 * d : 0.12 + 0.019 * d) *
                          (kind == KNM_KERNEL_GAUSSIAN ? 1.0 : 1.6);
        stage_us = 1.0e-6 * ps * (double)(g.stage * g.per_block) * 256.0 * per_cu;
    }
    const double slots = 256.0 * per_cu;
    // partials of more than 48 MB only where the compact rule has them too: the allocation-free call, whose scratch is
    // 64 MB, then cuts the stream the same way
    int64_t compact_len = 0;
    int64_t most = choose_chunks_compact(nF, nS, d, t, cross_term, kind, &compact_len);
    // sums that run through the chunk in fp32 are kept as short as the compact rule has them: in row sweeps of the
    // matrix-core reduction cut into 1 chunk in place of 16 the error of W against 64 bits went from 2.7e-7 to 3.1e-5
    // (n = 4.6M, M = 90k, 19 columns, v >= 0), and from 2.5e-7 to 4.4e-7 in U at n = 120k, M = 20k, 144 columns
    const bool fp32_sums = !gemm || (f16 ? gemm_f16_fp32_sums(d, t, kind) : gemm_fp32_sums(t));
    int64_t least = fp32_sums && !any_length && most > g.min_chunks ? most : g.min_chunks;
    if (parts && !any_length) {
        // no longer than the fp32 MFMA engine has them either: where it cut 3000 points into 6 chunks and this one would into 2 (d = 13, 120000 rows),
        // errors of W against 64 bits were up to 1.5 and of U up to 2 times those of that engine
        int64_t fp32_len = 0;
        const int64_t fp32_chunks = choose_chunks_by_time(nF, nS, d, t, cross_term, kind, false, false, &fp32_len);
        if (fp32_chunks > least) least = fp32_chunks;
    }
    const int64_t by_bytes = (int64_t)(((size_t)48 << 20) / (sizeof(float) * (size_t)nF * t));
    if (by_bytes > most) most = by_bytes;
    double best = 0.0;
    int64_t best_chunks = 0;
    auto consider = [&](int64_t chunks) {
        if (chunks > g.stages) chunks = g.stages;
        if (chunks > most) chunks = most;
        if (chunks < least) chunks = least;
        const int64_t len = (g.stages + chunks - 1) / chunks; // stages per chunk
        chunks = (g.stages + len - 1) / len;
        if (chunks == best_chunks || chunks > 65535) return;
        const double w = (double)(g.blocks * chunks);
        const double rounds = floor(w / slots), rest = w - rounds * slots;
        const double load = rounds + uneven + (rest == 0.0 ? 0.0 : per_cu > 1 && rest <= 256.0 ? 0.5 : 1.0);
        double us = load * ((double)len * stage_us) + (rounds + (rest > 0.0 ? 1.0 : 0.0)) * wg_us;
        if (gemm && w > 256.0) {
            double loss = chunks < 8 ? 0.55 - 0.055 * (double)chunks : 0.18 * (double)(chunks % 8) / (double)chunks;
            if (len > 64) loss += 0.02 * log2((double)len / 64.0);
            us *= 1.0 + loss * (d < 784 ? (double)d / 784.0 : 1.0);
        }
        if (chunks > 1) us += 3.0 + 1.0e-6 * (double)chunks * (double)nF * (double)t * 4.0 / 2.0;
        if (best_chunks == 0 || us < best) {
            best = us;
            best_chunks = chunks;
        }
    };
    consider(1);
    if ((double)g.blocks < 32.0 * slots) {
        for (int k = 2; k <= 16; ++k) consider(k);
        for (int k = 1; k <= 16; ++k) consider((int64_t)((double)k * slots / (double)g.blocks));
        if (gemm)
            for (int k = 24; k <= 128; k += 8) consider(k);
    }
    if (best_chunks == 0) best_chunks = least; // more than 65535 chunks: the sweep refuses them
    int64_t len = (g.stages + best_chunks - 1) / best_chunks;
    *chunk_len = len * g.stage;
    return (g.stages + len - 1) / len;
}

static bool three_parts(int64_t nF, int64_t nS, int d, int t, int cross_term, int kind)
{
    return cross_term != KNM_CROSS_F16X3 && packs_images(nF, nS, d, t, cross_term, kind);
}
int64_t choose_chunks_for(int64_t nF, int64_t nS, int d, int t, int cross_term, int kind, bool parts, int64_t *chunk_len)
{
    return choose_chunks_by_time(nF, nS, d, t, cross_term, kind, false, parts, chunk_len);
}
int64_t choose_chunks(int64_t nF, int64_t nS, int d, int t, int cross_term, int kind, int64_t *chunk_len)
{
    return choose_chunks_for(nF, nS, d, t, cross_term, kind, three_parts(nF, nS, d, t, cross_term, kind), chunk_len);
}

static bool bad_geom(const void *X, int64_t n, int d, int64_t ldx, const void *C, int64_t M, int64_t ldc,
                     float sigma, int t)
{
    return !X || !C || n <= 0 || M <= 0 || d <= 0 || t <= 0 || ldx < d || ldc < d || !(sigma > 0.0f);
}

// Common shift of a sweep's two point sets: mu[k] = mean of feature k over `rows` rows of P taken `stride` rows apart (a sample
// spread over the whole set, so that data stored in some order still gives a representative centre; it only has to
// be near the middle of the data).  It is kept only where it pays: if the mean itself is within sigma of the origin
// (|mu|^2 / 2 sigma^2 <= 0.5) the norm terms are small anyway, and mu is set to zero, which leaves the
// points exactly as they are (data with many exact zeros keeps them: the matrix cores draw less
// power on such operands, and the sweep runs measurably faster).
// Workgroup (x, y): features [x << fbits, ...), 256 >> fbits row lanes over row group y; fp64 partials, which the last
// workgroup to finish (`done` counts and wraps to zero) adds up in a fixed order.  Bound by the latency of its loads: 5 us for
// 1000 rows of 8 features, 9 us for 10000, 11 us for 16384 of 28, 40 us for 10000 of 784 (two launches and one
// workgroup per 32 features before: 4, 16, 46 and 30 us; the partials' sum without loads in flight and up to 1600 workgroups
// at the counter: 161 us for the last).
constexpr int64_t kMeanSample = 16384; // rows of the sample at most
constexpr int kMeanGroups = 64;       // row groups at most
__global__ __launch_bounds__(256) void column_shift_kernel(const float *__restrict__ P, int rows, int64_t stride, int64_t ld, int d,
                                                          float inv2s2, int fbits, double *__restrict__ part, unsigned *__restrict__ done,
                                                          float *__restrict__ mu)
{
    __shared__ double sh[256];
    __shared__ bool last;
    const int tid = threadIdx.x;
    const int f = tid & ((1 << fbits) - 1), rl = tid >> fbits, lanes = 256 >> fbits;
    const int k = (blockIdx.x << fbits) + f;
    const int groups = gridDim.y;
    const int per = (rows + groups - 1) / groups;
    const int r1 = (int)(blockIdx.y + 1) * per < rows ? (int)(blockIdx.y + 1) * per : rows;
    double s = 0.0;
    if (k < d) {
        const float *col = P + k;
        const int64_t step = stride * ld;
        int r = (int)blockIdx.y * per + rl;
        for (; r + 3 * lanes < r1; r += 4 * lanes) {
            const float a0 = col[r * step], a1 = col[(r + lanes) * step];
            const float a2 = col[(r + 2 * lanes) * step], a3 = col[(r + 3 * lanes) * step];
            s += ((double)a0 + (double)a1) + ((double)a2 + (double)a3);
        }
        for (; r < r1; r += lanes) s += (double)col[r * step];
    }
    sh[tid] = s;
    __syncthreads();
    if (rl == 0 && k < d) {
        for (int i = 1; i < lanes; ++i) s += sh[(i << fbits) + f];
        part[(int64_t)blockIdx.y * d + k] = s;
    }
    __threadfence();
    __syncthreads();
    if (tid == 0) last = atomicInc(done, gridDim.x * gridDim.y - 1) == gridDim.x * gridDim.y - 1;
    __syncthreads();
    if (!last) return;
    __threadfence();
    double sq = 0.0;
    for (int c = tid; c < d; c += 256) {
        double total = 0.0;
#pragma unroll 16
        for (int y = 0; y < groups; ++y) total += part[(int64_t)y * d + c];
        const float m = (float)(total / (double)rows);
        const float v = (m == m && fabsf(m) < 3.0e38f) ? m : 0.0f; // a NaN or Inf in the data must not spread to every point
        mu[c] = v;
        sq += (double)v * (double)v;
    }
    sh[tid] = sq;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (tid < w) sh[tid] += sh[tid + w];
        __syncthreads();
    }
    const bool keep = sh[0] * (double)inv2s2 > 0.5;
    if (!keep)
        for (int c = tid; c < d; c += 256) mu[c] = 0.0f;
    if (tid == 0) mu[d] = keep ? 1.0f : 0.0f; // lets the hot loops skip the loads of an all-zero shift
}
// mu_buf: the shift and its flag, then (8-byte aligned) the partials
static int mean_feature_bits(int d) { return d <= 8 ? 3 : d <= 16 ? 4 : 5; }
static int mean_feature_groups(int d) { return (d + (1 << mean_feature_bits(d)) - 1) >> mean_feature_bits(d); }
static int mean_groups(int64_t rows, int d)
{
    int64_t g = (rows + 63) / 64;
    if (g > kMeanGroups) g = kMeanGroups;
    // at most 256 workgroups: each pays for a fence and a turn at the counter
    const int most = 256 / mean_feature_groups(d);
    return g > most ? (most > 0 ? most : 1) : (int)g;
}
static size_t mu_offset(int d) { return (sizeof(float) * ((size_t)d + 1) + 7) & ~(size_t)7; }
static size_t mu_bytes_wanted(int64_t rows, int d)
{
    return mu_offset(d) + sizeof(double) * (size_t)mean_groups(rows < kMeanSample ? rows : kMeanSample, d) * d;
}
static int column_shift(knm_ctx *ctx, const float *P, int64_t rows, int64_t ld, int d, float sigma, float *mu)
{
    const int64_t stride = (rows + kMeanSample - 1) / kMeanSample; // every stride-th row, spread over the set
    const int sample = (int)((rows + stride - 1) / stride);
    double *part = reinterpret_cast<double *>(reinterpret_cast<char *>(mu) + mu_offset(d));
    hipLaunchKernelGGL(column_shift_kernel, dim3((unsigned)mean_feature_groups(d), (unsigned)mean_groups(sample, d)), dim3(256),
                       0, ctx->stream, P, sample, stride, ld, d, 1.0f / (2.0f * sigma * sigma), mean_feature_bits(d), part, ctx->range_count + 32, mu);
    return hipGetLastError() == hipSuccess ? KNM_OK : fail(ctx, KNM_HIP_ERROR, "column_shift_kernel launch");
}

SweepShare::SweepShare(knm_ctx *c, const float *X, int64_t n_, int64_t ldx, const float *C, int64_t M, int64_t ldc, int d_, float sigma_,
                       int t_, bool pooled_)
    : ctx(c), P{X, C}, n{n_, M}, ld{ldx, ldc}, d(d_), sigma(sigma_), t(t_), shift_P(M <= n_ ? C : X), shift_n(M <= n_ ? M : n_),
      shift_ld(M <= n_ ? ldc : ldx), pooled(pooled_)
{
    // (an unregistered block is only one that is not given up)
    if (pooled) (void)(spare_add(ctx, 0, &keep) && spare_add(ctx, 1, &img[0]) && spare_add(ctx, 1, &img[1]));
}
SweepShare::~SweepShare()
{
    if (pooled) {
        spare_remove(ctx, 0, &keep);
        for (void *&p : img) spare_remove(ctx, 1, &p);
        for (void *p : {img[0], img[1], keep})
            if (p) pool_give(ctx, p);
    }
    if (ctx->mu_owner == this) ctx->mu_owner = nullptr;
}

// Points the kept image of set k must have room for: as fixed points whole fixed blocks, as stream points whole chunks.
static int64_t share_rows(const int64_t (&n)[2], int k, int d, int t, int cross_term, int kind)
{
    int64_t len = 0;
    const int64_t chunks = choose_chunks(n[k ^ 1], n[k], d, t, cross_term, kind, &len);
    const int64_t fixed = (n[k] + gemm_fixed_per_block() - 1) / gemm_fixed_per_block() * gemm_fixed_per_block();
    return chunks * len > fixed ? chunks * len : fixed;
}
constexpr size_t kShareCap = (size_t)8 << 30; // bytes of the kept images of a pair at most (unless the caller set a cap)

// Bytes of both images of a product's point sets on the K-loop split-fp16 engine, 0 if they are not kept
static size_t product_image_bytes(const int64_t (&n)[2], int d, int t, int kind, size_t limit)
{
    if (!use_gemm_engine(d, t, KNM_CROSS_F16X3, kind)) return 0;
    const size_t pp = gemm_f16_pack_bytes_per_point(d);
    const size_t bytes = pp * (size_t)(share_rows(n, 0, d, t, KNM_CROSS_F16X3, kind) + share_rows(n, 1, d, t, KNM_CROSS_F16X3, kind));
    return bytes <= (limit ? limit : kShareCap) ? bytes : 0;
}

// Decides, at the first sweep of a scope (and again if the arithmetic changed), whether images are kept, and finds room for
// them: a fit's in blocks of the pool, a product's in the context's image workspace behind the head.
static int share_images(knm_ctx *ctx, SweepShare *sh)
{
    if (sh->decided && sh->cross_term == ctx->cross_term && sh->kind == ctx->kernel_kind) return KNM_OK;
    for (int k = 0; k < 2; ++k) {
        if (sh->img[k] && sh->pooled) pool_give(ctx, sh->img[k]);
        sh->img[k] = nullptr;
        sh->rows[k] = sh->ready[k] = 0;
    }
    if (sh->keep && sh->pooled) pool_give(ctx, sh->keep);
    sh->keep = nullptr;
    sh->keep_decided = false;
    sh->decided = true;
    sh->cross_term = ctx->cross_term;
    sh->kind = ctx->kernel_kind;
    if (!packs_images(sh->n[0], sh->n[1], sh->d, sh->t, ctx->cross_term, ctx->kernel_kind) || ctx->static_mode) return KNM_OK;
    const bool gemm = use_gemm_engine(sh->d, sh->t, ctx->cross_term, ctx->kernel_kind);
    if (!gemm && !sh->pooled) return KNM_OK;
    const size_t pp = image_bytes_per_point(sh->d, sh->t, ctx->cross_term, ctx->kernel_kind);
    const int64_t r0 = share_rows(sh->n, 0, sh->d, sh->t, ctx->cross_term, ctx->kernel_kind);
    const int64_t r1 = share_rows(sh->n, 1, sh->d, sh->t, ctx->cross_term, ctx->kernel_kind);
    if (pp * (size_t)(r0 + r1) > (ctx->pack_limit ? ctx->pack_limit : kShareCap)) return KNM_OK;
    if (sh->pooled) {
        for (int k = 0; k < 2; ++k)
            if (pool_take(ctx, pp * (size_t)(k == 0 ? r0 : r1), &sh->img[k],
                          ctx->cross_term == KNM_CROSS_F16X3 ? PoolUse::kOptional : PoolUse::kForSpeed) != hipSuccess) {
                // no room: the sweeps pack slab by slab (or not at all)
                if (sh->img[0]) pool_give(ctx, sh->img[0]);
                sh->img[0] = sh->img[1] = nullptr;
                return KNM_OK;
            }
    } else {
        const size_t head = gemm_f16_head_bytes();
        int st = ensure(ctx, &ctx->pack_buf, &ctx->pack_bytes, head + pp * (size_t)(r0 + r1));
        if (st) return st;
        sh->img[0] = reinterpret_cast<char *>(ctx->pack_buf) + head;
        sh->img[1] = static_cast<char *>(sh->img[0]) + pp * (size_t)r0;
    }
    sh->rows[0] = r0;
    sh->rows[1] = r1;
    return KNM_OK;
}

// sigma as the engines take it.  Kernels of r = |x - c|: with sigma / (c sqrt(2 log2 e)) in place of sigma the engines'
// accumulators hold -(log2(e) c r / sigma)^2, whose root the kernel takes before the exp2
// (c = 1 Laplacian, sqrt(3) and sqrt(5) for the two Matern kernels)
static float engine_sigma(float sigma, int kind)
{
    const float c_kind = kind == KNM_KERNEL_MATERN32 ? 1.7320508075688772f : kind == KNM_KERNEL_MATERN52 ? 2.23606797749979f : 1.0f;
    return kind == KNM_KERNEL_GAUSSIAN ? sigma : sigma / (c_kind * sqrtf(2.0f * 1.4426950408889634f));
}

constexpr size_t kKeepCap = (size_t)8 << 30; // bytes of a fit's kept kernel values at most

// Whether `uses` sweeps over n x M kernel values take less time with the values formed once and read by each.  Estimates in ps per
// value, measured at n = 300k, M = 20k: a sweep 0.62 (d = 100), 1.06 (200), 1.53 (300), 3.8 (784), one with 10 columns 0.76, 1.23, 1.79
// and 4.2, up to a fifth less on data with many zeros; reading 0.75 (5.4 TB/s), 1.25 with 17 to 32 columns.  Fits with n =
// 60k, M = 10k, 10 iterations: with 1 column 0.965 times as fast at d = 100, 1.003 at 130, 1.085 at 200, 1.44 at 500; with 10 columns 1.01,
// 1.05, 1.11 and 1.48; with 24 columns 0.92, 0.95, 1.00 and 1.29; the fp32 engine 1.36 at d = 70 and 1 column, 2.1 at d = 200 and 24.
// Values that do not stay in the caches (64 MB and more) have 16 us a sweep more, the readers' launches and their uneven ends; without them in
// the estimate fits of 13000 x 3249, 30000 x 3000 and 40000 x 8000 at 20 iterations lost 4 to 7 % at d = 120 to 160 with 1 and 4 columns.
// Where reading and forming meet there: d = 190, 168 and 150 with 1 column, 200, 160 and 132 with 4; 133 and 120 at 150k x 9000.
static bool keeping_pays(int64_t n, int64_t M, int d, int t, int cross_term, int kind, int uses)
{
    if (t > kept_max_t() || !use_gemm_engine(d, t, cross_term, kind)) return false;
    const bool f16 = cross_term == KNM_CROSS_F16X3, mc = f16 && gemm_f16_matrix_reduction(d, t);
    const double values = 1.0e-6 * (double)n * (double)M; // us for 1 ps each
    const double read = values * (t <= 16 ? 0.75 : 1.25) + (values >= 16.0 ? 16.0 : 0.0);
    const double form = values * ((f16 ? 0.14 + 0.0045 * d : 0.2 + 0.02 * d) + (kind == KNM_KERNEL_GAUSSIAN ? 0.0 : 0.2));
    // (the matrix-core reduction has four launches more, which is most of a small sweep)
    const double sweep = form + values * (mc || t > 5 ? 0.15 : 0.02 * t) + (mc ? 15.0 : 0.0);
    return form + read * uses < sweep * uses;
}

// Rows of X whose kernel values a product keeps from its row sweep to its sums over the columns, 0 if it forms them twice: where a second
// sweep (estimated as in keeping_pays) takes longer than storing the values beside the first (0.2 ps per value) and reading them
// (0.8), and its sums are those of the vector ALU, which kept_rows_kernel repeats to the last bit.  The line lies at d = 260 with 1 column, 240
// with 4, 234 with 6 to 12.  Products as fast as by two sweeps, 1 column at d = 262, normal rows and rows of which four fifths are zeros (whose two
// sweeps take a fifth less, at a higher clock): 5000 x 500 1.14 and 1.15, 36099 x 2443 1.13 and 1.02, 100k x 1500 1.15 and 1.03, 50000 x 8000
// 1.27 and 1.10, 300k x 20k 1.27 and 1.13; 4 columns at d = 244 1.18, 1.14 and 1.03, 1.27 and 1.25, 1.23 and 1.11, 1.25 and 1.09; 8 columns
// at d = 236 1.20, 1.20 and 1.16, 1.29 and 1.20, 1.23 and 1.12, 1.26 and 1.12; d = 784 1.3 to 1.6.  (While values went through the caches as
// other data do, and pushed the operands out, 1 column at d = 262 was 0.96 to 1.10 and, on rows of zeros, 0.84 to 0.93 times as fast.)
// Slabs of 16 GiB were no faster than of 4.
// The more centres, the fewer rows has a slab, and each reads all centres again: 400k centres (2560 rows) 1.04, 1.07, 1.11 and 1.18 at d = 260,
// 280, 300 and 340 with 1 column, 1M centres (1024 rows) 1.00, 1.03, 1.04 and 1.12, 1.53 at d = 784; 4M centres (256 rows) 0.94 at d = 270,
// 1.14 at 400 and 0.74 at 784, where the centres' image is not kept either.
constexpr size_t kKeepSlabCap = (size_t)4 << 30; // bytes of a slab at most
constexpr int64_t kKeepSlabRows = 1024;          // rows of a slab at least, where there are several
// More columns than those take the values from memory for both sums (prod_kept_many).  In ps per value at 120k x 20k: forming and storing
// 0.15 + 0.0046 d, a sum of up to 32 columns 0.85, 64 0.95, 128 1.2, 160 1.45, against two sweeps of 0.27 + 0.0047 d, 0.45 + 0.0047 d,
// 0.75 + 0.0055 d and 1.05 + 0.0061 d: they meet at d = 293, 260, 180 and 140.  The lines lie beyond, for rows of zeros, whose sweeps are up to a
// fifth faster, and for few centres, whose launches and partials count: 13 columns at d = 320 1.14 times as fast at 200k x 8000 and 0.96 with rows of
// zeros, 0.94 and 0.87 at 300k x 500; above the lines 1.06 to 1.36 at the line, 1.25 to 1.58 with 30 columns at d = 784, 1.7 to 2 with 200 at 440.
// Only where the sweeps' own sums run on the matrix cores, in every launch: 13 to 16 columns from 337 to 401 features on, and what a multiple of 160
// leaves, are summed by the vector ALU there, without the halves of values and vectors, and this kernel's sums are up to 1.7 (W) and 4.2 (U) times
// as far from 64 bits (d = 450, 13 columns; d = 784, 16); with matrix-core sums on both sides 0.99 to 1.01 times.
static bool keeping_many_pays(int64_t n, int64_t M, int d, int t)
{
    const int least = t <= 32 ? 450 : t <= 64 ? 320 : t <= 128 ? 210 : 180;
    const int last = (t - 1) % kept_many_max_t() + 1; // columns of the last launch
    return t > kept_rows_max_t() && d >= least && gemm_f16_matrix_reduction(d, last) && (double)n * (double)M >= 1.0e8;
}
static int64_t product_keep_rows(int64_t n, int64_t M, int d, int t, int cross_term, int kind)
{
    if (cross_term != KNM_CROSS_F16X3 || kind != KNM_KERNEL_GAUSSIAN || !use_gemm_engine(d, t, cross_term, kind)) return 0;
    if (t > kept_rows_max_t() ? !keeping_many_pays(n, M, d, t)
                              : gemm_f16_matrix_reduction(d, t) || 0.14 + 0.0045 * d + (t > 5 ? 0.15 : 0.03 * t) < 1.34)
        return 0;
    int64_t rows = n;
    if (kept_bytes(n, M) > kKeepSlabCap) {
        rows = (int64_t)(kKeepSlabCap / kept_bytes(256, M)) * 256;
        if (rows >= 16384) rows = rows / 16384 * 16384; // 64 fixed blocks x 8 chunks fill the chip
        if (rows < kKeepSlabRows) return 0;
    }
    return rows;
}

// How prod_kept_many cuts the sums over `in` points for `out` results, and its workspace.  The fp32 sums run over as many points as
// those of the engine's sweeps (over all points, `in_all`), or fewer where that fills the chip's 256 places better: the least of rounds x
// stages of 64 points (0.35 us and 0.3 per 32 columns each, 4 us a workgroup) and the partials' way to memory and back.
static int64_t many_chunk(int64_t in, int64_t out, int64_t in_all, int d, int t)
{
    int64_t longest = 0;
    (void)choose_chunks(out, in_all, d, t, KNM_CROSS_F16X3, KNM_KERNEL_GAUSSIAN, &longest);
    const int64_t tiles = (in + 127) / 128, blocks = (out + 255) / 256, least = (tiles * 128 + longest - 1) / longest;
    const double stage_us = 0.35 + 0.3 * (double)((t < kept_many_max_t() ? t : kept_many_max_t()) + 31) / 32.0;
    int64_t best = 0;
    double best_us = 0.0;
    for (int64_t c = least; c <= 3 * least + 16 && c <= tiles; ++c) {
        const int64_t len = (tiles + c - 1) / c, chunks = (tiles + len - 1) / len;
        const int64_t rounds = (blocks * chunks + 255) / 256;
        const double us = (double)rounds * (2.0 * (double)len * stage_us + 4.0) + 1.6e-6 * (double)chunks * (double)out * (double)t;
        if (best == 0 || us < best_us) {
            best = len;
            best_us = us;
        }
    }
    return best * 128;
}
struct ManyPlan {
    int64_t row_chunk, col_chunk;   // points per chunk of the sums over the centres, over a slab's rows
    int64_t row_chunks, col_chunks; // at most
    int group;                      // columns per launch
    size_t at[7], bytes;
    ManyPlan(int64_t n, int64_t rows, int64_t M, int d, int t)
    {
        group = t < kept_many_max_t() ? t : kept_many_max_t();
        row_chunk = many_chunk(M, rows, M, d, t);
        col_chunk = many_chunk(rows, M, n, d, t);
        row_chunks = (M + row_chunk - 1) / row_chunk;
        col_chunks = (rows + col_chunk - 1) / col_chunk;
        auto padded = [](int64_t n) { return (n + 127) / 128 * 128; };
        // values, partials of W and of U, running U, images of V and W, their columns' scales
        const size_t pieces[7] = {kept_bytes(rows, M), sizeof(float) * (size_t)row_chunks * (size_t)rows * t,
                                  sizeof(float) * (size_t)col_chunks * (size_t)M * t, sizeof(double) * (size_t)M * t,
                                  vector_image_bytes(group, padded(M)), vector_image_bytes(group, padded(rows)), 2 * gemm_f16_head_bytes()};
        bytes = 0;
        for (int i = 0; i < 7; ++i) {
            at[i] = bytes;
            bytes += (pieces[i] + 255) & ~(size_t)255;
        }
    }
};

// Forms the kernel values of set f against set s into `keep` (the images of both sets are there).
static int form_values(knm_ctx *ctx, SweepShare *sh, int f, int s, const float *mu, float *keep)
{
    SweepArgs a{};
    a.F = sh->P[f]; a.nF = sh->n[f]; a.ldf = sh->ld[f];
    a.S = sh->P[s]; a.nS = sh->n[s]; a.lds = sh->ld[s];
    a.d = sh->d;
    a.mu = mu;
    a.range_count = ctx->range_count;
    a.t = 1;
    a.kind = sh->kind;
    a.sigma = engine_sigma(sh->sigma, sh->kind);
    a.n_chunks = choose_chunks(a.nF, a.nS, a.d, 1, sh->cross_term, sh->kind, &a.chunk_len);
    a.fimg = sh->img[f];
    a.simg = sh->img[s];
    a.fimg_ready = sh->ready[f] >= kept_rows(sh->n[f]);
    a.simg_ready = f == s || sh->ready[s] >= kept_rows(sh->n[s]);
    a.keep = keep;
    a.keep_s32 = kept_stream_blocks(a.nS);
    for (int k : {f, s})
        if (sh->ready[k] < kept_rows(sh->n[k])) sh->ready[k] = kept_rows(sh->n[k]);
    const hipError_t e = sh->cross_term == KNM_CROSS_F16X3 ? launch_keep_f16(a, ctx->stream) : launch_sweep_gemm(a, ctx->stream);
    return e == hipSuccess ? KNM_OK : fail(ctx, KNM_HIP_ERROR, "forming kernel values", e);
}

// Decides, at a pair's first sweep, whether its kernel values are kept, and forms them.
static int keep_values(knm_ctx *ctx, SweepShare *sh, int f, int s, bool column_sweep, const float *mu)
{
    const bool f16 = sh->cross_term == KNM_CROSS_F16X3;
    const bool ready = !f16 || (sh->img[0] != nullptr && sh->rows[f] >= kept_rows(sh->n[f]) && sh->rows[s] >= kept_rows(sh->n[s]));
    if (sh->keep_decided || sh->uses == 0 || !sh->pair(f, s)) return KNM_OK;
    sh->keep_decided = true;
    const size_t bytes = kept_bytes(sh->n[f], sh->n[s]);
    if (bytes > kKeepCap || !ready || !keeping_pays(sh->n[f], sh->n[s], sh->d, sh->t, sh->cross_term, sh->kind, sh->uses)) return KNM_OK;
    if (!f16 && (!gemm_leading_dimension_ok(sh->ld[f]) || !gemm_leading_dimension_ok(sh->ld[s]))) return KNM_OK;
    void *p = nullptr;
    if (pool_take(ctx, bytes, &p, PoolUse::kForSpeed) != hipSuccess) return KNM_OK; // no room: the sweeps form the values
    sh->keep = p;
    sh->keep_columns = column_sweep;
    sh->keep_n[0] = sh->n[f];
    sh->keep_n[1] = sh->n[s];
    return form_values(ctx, sh, f, s, mu, static_cast<float *>(p));
}

static void drop_slab(knm_ctx *ctx)
{
    if (ctx->slab == nullptr) return;
    spare_remove(ctx, 0, &ctx->slab);
    pool_drop(ctx, ctx->slab);
    ctx->slab = nullptr;
}

// The context's slab for as long as a product uses it: `bytes` of it, or none.  A call on a stream that is being captured takes what is
// there and allocates nothing, and what it took stays until the context outgrows it or its workspace is released, as the other buffers of a
// captured product do.
struct SlabUse {
    knm_ctx *ctx;
    void *p = nullptr;
    SlabUse(knm_ctx *c, size_t bytes) : ctx(c)
    {
        const bool capturing = is_capturing(ctx);
        if (ctx->slab == nullptr || ctx->slab_bytes < bytes) {
            if (capturing) return;
            drop_slab(ctx);
            bytes = (bytes + 255) & ~(size_t)255;
            if (pool_take(ctx, bytes, &ctx->slab, PoolUse::kForSpeed) != hipSuccess) return;
            ctx->slab_bytes = pool_bytes(ctx, ctx->slab);
            ctx->slab_captured = false;
        }
        spare_remove(ctx, 0, &ctx->slab);
        ctx->slab_captured |= capturing;
        p = ctx->slab;
    }
    ~SlabUse()
    {
        // (an unregistered block is only one that is not given up)
        if (p != nullptr && !ctx->slab_captured) (void)spare_add(ctx, 0, &ctx->slab);
    }
    SlabUse(const SlabUse &) = delete;
    SlabUse &operator=(const SlabUse &) = delete;
};

// The sums over kept values `keep` of nF fixed and nS stream points, `part` holding kept_chunks() partials of n_out x t.
static int kept_partials(knm_ctx *ctx, const float *keep, int64_t nF, int64_t nS, bool over_stream, const float *vec, const float *wgt,
                         int t, double *part, int chunks)
{
    KeptArgs k{};
    k.values = keep;
    k.nF = nF;
    k.nS = nS;
    k.over_stream = over_stream;
    k.vec = vec;
    k.t = t;
    k.wgt = wgt;
    k.part = part;
    k.chunks = chunks;
    const hipError_t e = launch_kept_sum(k, ctx->stream);
    return e == hipSuccess ? KNM_OK : fail(ctx, KNM_HIP_ERROR, "launch_kept_sum", e);
}

// Bytes of the packed-operand workspace one sweep that packs images asks for: the same rule for the sweep itself and for
// knm_workspace_bytes.  `limit` = the caller's cap, 0 for the defaults.
static size_t pack_bytes_wanted(int64_t nF, int d, int t, int cross_term, int kind, size_t limit, int64_t chunks, int64_t chunk_len)
{
    if (use_gemm_engine(d, t, cross_term, kind)) {
        // packed images of both operands: whole if they fit 8 GiB, else the smaller one
        // whole and the other in slabs
        const size_t per_point = gemm_f16_pack_bytes_per_point(d);
        const int64_t nFp = (nF + gemm_fixed_per_block() - 1) / gemm_fixed_per_block() * gemm_fixed_per_block();
        size_t want = gemm_f16_head_bytes() + per_point * (size_t)(nFp + chunks * chunk_len); // head + both images
        const size_t cap = limit ? limit : (size_t)8 << 30;
        const size_t least = gemm_f16_min_pack_bytes(nF, chunks * chunk_len, chunk_len, d);
        if (want > cap) want = cap;
        if (want < least) want = least;
        return want;
    }
    // packed image of the stream points: all of it, or slabs of at most 2 GiB
    const size_t per_point = image_bytes_per_point(d, t, cross_term, kind);
    size_t want = per_point * (size_t)(chunks * chunk_len);
    const size_t cap = limit ? limit : (size_t)2 << 30;
    if (want > cap) want = (cap / (per_point * chunk_len) + 1) * per_point * chunk_len;
    return want;
}

// out[f, c] = sum_s k(F_f, S_s) vec[s, c] wgt[s]  for c < t (all arrays leading dimension t); the
// result goes to `out` (fp32) or, if that is null, to `out64`: then the chunk partials of the K-loop
// engines stay in fp64 from the kernels' running sums to the merged result
static int sweep(knm_ctx *ctx, const float *F, int64_t nF, int64_t ldf, const float *S, int64_t nS, int64_t lds,
                 int d, float sigma, const float *vec, const float *wgt, int t, float *out, double *out64,
                 hipEvent_t after_sweep, bool column_sweep)
{
    int64_t chunk_len = 0;
    int64_t chunks = choose_chunks(nF, nS, d, t, ctx->cross_term, ctx->kernel_kind, &chunk_len);
    // the engine that has fp32 numbers in three parts takes the sweep, unless there is no room for its image
    bool parts = three_parts(nF, nS, d, t, ctx->cross_term, ctx->kernel_kind);
    if (ctx->static_mode) {
        // where these partials and the least operand images do not fit the scratch together: fewer chunks; the fp32 MFMA engine takes
        // the sweep, cut as it would be without the other engine, where an image of three-part numbers does not fit whatever the chunks
        auto fits = [&] {
            const size_t least = !parts && ctx->cross_term != KNM_CROSS_F16X3 ? 0
                                 : use_gemm_engine(d, t, ctx->cross_term, ctx->kernel_kind)
                                     ? gemm_f16_min_pack_bytes(nF, chunks * chunk_len, chunk_len, d)
                                     : image_bytes_per_point(d, t, ctx->cross_term, ctx->kernel_kind) * (size_t)chunk_len;
            return sizeof(float) * (size_t)chunks * nF * t + mu_bytes_wanted(kMeanSample, d) + least + 1024 <= kStaticScratchBytes;
        };
        auto choose = [&] {
            chunks = choose_chunks_for(nF, nS, d, t, ctx->cross_term, ctx->kernel_kind, parts, &chunk_len);
            if (!fits()) chunks = choose_chunks_compact(nF, nS, d, t, ctx->cross_term, ctx->kernel_kind, &chunk_len);
            if (!fits()) chunks = choose_chunks_by_time(nF, nS, d, t, ctx->cross_term, ctx->kernel_kind, true, parts, &chunk_len);
            if (!fits()) chunks = choose_chunks_compact(nF, nS, d, t, ctx->cross_term, ctx->kernel_kind, &chunk_len); // refused below
            return fits();
        };
        if (!choose() && parts) {
            parts = false;
            (void)choose();
        }
    }
    if (chunks > 65535) return fail(ctx, KNM_UNSUPPORTED, "too many stream chunks");
    const bool gemm = use_gemm_engine(d, t, ctx->cross_term, ctx->kernel_kind);
    if (gemm && ctx->cross_term == KNM_CROSS_F32 && (!gemm_leading_dimension_ok(ldf) || !gemm_leading_dimension_ok(lds)))
        return fail(ctx, KNM_UNSUPPORTED, "leading dimension above 5.5 million elements in the fp32-MFMA K-loop engine");
    const bool part_is_64 = out64 != nullptr && gemm;
    const bool merged = chunks > 1 || out64 != nullptr; // an fp64 result is always written by the merge pass
    if (ctx->static_mode) ctx->static_used = 0; // every sweep carves its pieces afresh
    float *part = nullptr;
    // common shift of the two sets, from the smaller one of them (or of the pair they belong to)
    SweepShare *sh = ctx->static_mode ? nullptr : ctx->share;
    const int set_f = sh ? sh->which(F, nF, ldf) : -1, set_s = sh ? sh->which(S, nS, lds) : -1;
    const bool shared = set_f >= 0 && set_s >= 0 && sh->d == d && sh->sigma == sigma;
    float *mu = nullptr;
    {
        const bool from_f = nF <= nS;
        const float *P = from_f ? F : S;
        int64_t rows = from_f ? nF : nS, ld = from_f ? ldf : lds;
        if (shared) {
            P = sh->shift_P;
            rows = sh->shift_n;
            ld = sh->shift_ld;
        }
        int st = acquire(ctx, &ctx->mu_buf, &ctx->mu_bytes, mu_bytes_wanted(rows, d), &mu);
        if (st) return st;
        if (!shared || ctx->mu_owner != sh) {
            st = column_shift(ctx, P, rows, ld, d, sigma, mu);
            if (st) return st;
            if (!ctx->static_mode) ctx->mu_owner = shared ? sh : nullptr;
        }
    }
    if (shared) {
        int st = share_images(ctx, sh);
        if (!st) st = keep_values(ctx, sh, set_f, set_s, column_sweep, mu);
        if (st) return st;
        const bool over_stream = column_sweep == sh->keep_columns;
        const int64_t kF = over_stream ? nF : nS, kS = over_stream ? nS : nF;
        if (sh->keep && sh->pair(set_f, set_s) && kF == sh->keep_n[0] && kS == sh->keep_n[1] && t <= kept_max_t()) {
            const int parts = kept_chunks(kF, kS, over_stream, t);
            st = acquire(ctx, &ctx->part_buf, &ctx->part_bytes, sizeof(double) * (size_t)parts * nF * t, &part);
            if (st) return st;
            if (sh->keep) { // (not given up for the partials)
                double *part64 = reinterpret_cast<double *>(part);
                st = kept_partials(ctx, static_cast<float *>(sh->keep), kF, kS, over_stream, vec, wgt, t, part64, parts);
                if (st) return st;
                if (after_sweep) (void)hipEventRecord(after_sweep, ctx->stream);
                const hipError_t e = launch_merge(nullptr, part64, parts, nF * t, 1, out64 != nullptr ? nullptr : out, out64, 1, nF * t, ctx->stream);
                return e == hipSuccess ? KNM_OK : fail(ctx, KNM_HIP_ERROR, "launch_merge", e);
            }
        }
    }
    if (merged) {
        int st = acquire(ctx, &ctx->part_buf, &ctx->part_bytes,
                         (part_is_64 ? sizeof(double) : sizeof(float)) * (size_t)chunks * nF * t, &part);
        if (st) return st;
    }
    // columns per launch
    int group = 1;
    for (int c = 0; c < t; c += group) {
        // (K-loop split-fp16 engine: wide launches when the vectors can be given as a packed image, which a
        // call that must not allocate does without, as does one whose image would be very large)
        bool vector_image = gemm && ctx->cross_term == KNM_CROSS_F16X3 && !ctx->static_mode;
        if (vector_image) {
            const int wide = gemm_f16_group_t(d, t - c, ctx->kernel_kind, true);
            vector_image = gemm_f16_vector_image_bytes(d, t - c < wide ? t - c : wide, chunks * chunk_len) <= kVectorImageCap;
        }
        group = !gemm ? 1 : (ctx->cross_term == KNM_CROSS_F16X3 ? gemm_f16_group_t(d, t - c, ctx->kernel_kind, vector_image) : gemm_max_t());
        SweepArgs a;
        a.F = F; a.nF = nF; a.ldf = ldf;
        a.S = S; a.nS = nS; a.lds = lds;
        a.d = d;
        a.mu = mu;
        a.range_count = ctx->range_count;
        a.vec = vec + c; a.ldv = t;
        a.t = (t - c < group) ? t - c : group;
        a.wgt = wgt;
        a.out = merged ? part + c : out + c;
        a.out64 = part_is_64 ? reinterpret_cast<double *>(part) + c : nullptr;
        a.ldo = t;
        a.chunk_stride = nF * t;
        a.chunk_len = chunk_len;
        a.n_chunks = chunks;
        a.kind = ctx->kernel_kind;
        a.sigma = engine_sigma(sigma, a.kind);
        if (shared && sh->slab != nullptr) { // (kept_rows_max_t() columns are one launch)
            a.keep = sh->slab;
            a.keep_s32 = kept_stream_blocks(nS);
        }
        const bool f16 = !gemm && ctx->cross_term == KNM_CROSS_F16X3 && d <= f16_max_d();
        hipError_t e;
        // packed operands of the split-fp16 engines: what the engine would like, or (static scratch)
        // as many whole slabs as the rest of the scratch holds; the same region serves every column group
        auto pack_room = [&](size_t *want) -> int {
            *want = pack_bytes_wanted(nF, d, t, ctx->cross_term, ctx->kernel_kind, ctx->pack_limit, chunks, chunk_len);
            if (!ctx->static_mode) return KNM_OK;
            const size_t at = (ctx->static_used + 255) & ~(size_t)255;
            const size_t room = at < kStaticScratchBytes ? kStaticScratchBytes - at : 0;
            if (gemm) {
                const size_t least = gemm_f16_min_pack_bytes(nF, chunks * chunk_len, chunk_len, d);
                if (*want > room) *want = room;
                if (*want < least) *want = least; // acquire() then reports that it does not fit
            } else {
                const size_t per_chunk = image_bytes_per_point(d, t, ctx->cross_term, ctx->kernel_kind) * (size_t)chunk_len;
                const size_t fit = room / per_chunk * per_chunk;
                if (*want > fit) *want = fit > 0 ? fit : per_chunk;
            }
            return KNM_OK;
        };
        float *pack = nullptr;
        const size_t mark_used = ctx->static_used;
        const int64_t f_rows = (nF + gemm_fixed_per_block() - 1) / gemm_fixed_per_block() * gemm_fixed_per_block();
        const int64_t s_rows = chunks * chunk_len;
        bool kept = shared && sh->img[0] != nullptr && sh->rows[set_s] >= s_rows && (!gemm || sh->rows[set_f] >= f_rows);
        auto use_images = [&] {
            a.simg = sh->img[set_s];
            a.simg_ready = sh->ready[set_s] >= s_rows;
            if (!a.simg_ready) sh->ready[set_s] = s_rows;
            if (gemm) {
                a.fimg = sh->img[set_f];
                a.fimg_ready = sh->ready[set_f] >= f_rows;
                if (!a.fimg_ready) sh->ready[set_f] = f_rows;
            }
        };
        if (gemm && ctx->cross_term == KNM_CROSS_F16X3) {
            size_t want = gemm_f16_head_bytes();
            int st = kept ? KNM_OK : pack_room(&want);
            if (!st) st = acquire(ctx, &ctx->pack_buf, &ctx->pack_bytes, want, &pack);
            if (st) return st;
            // the vectors as a packed image, when the matrix-core reduction runs and the image is of moderate
            // size (a call that must not allocate leaves the conversion to the workgroups)
            const size_t vbytes = vector_image ? gemm_f16_vector_image_bytes(d, a.t, chunks * chunk_len) : 0;
            if (vbytes > 0) {
                st = ensure(ctx, &ctx->vimg_buf, &ctx->vimg_bytes, vbytes);
                if (st) return st;
                a.vimg = ctx->vimg_buf;
            }
            if (kept && (sh->img[0] == nullptr || sh->img[1] == nullptr)) { // given up for one of these two
                kept = false;
                st = pack_room(&want);
                if (!st) st = acquire(ctx, &ctx->pack_buf, &ctx->pack_bytes, want, &pack);
                if (st) return st;
            }
            if (kept) use_images();
            e = launch_sweep_gemm_f16(a, pack, want, ctx->stream);
        } else if (gemm) {
            e = launch_sweep_gemm(a, ctx->stream);
        } else if (f16) {
            size_t want = 0;
            int st = KNM_OK;
            if (!kept) {
                st = pack_room(&want);
                if (!st) st = acquire(ctx, &ctx->pack_buf, &ctx->pack_bytes, want, &pack);
            }
            if (st) return st;
            if (kept) use_images();
            e = launch_sweep_f16(a, pack, want, ctx->stream);
        } else {
            // the image of three-part numbers is for speed alone: where the card has no room to spare for it the fp32 MFMA engine
            // takes the rows as they are
            size_t want = 0;
            if (parts && !kept) {
                int st = pack_room(&want);
                if (!st && ctx->static_mode) st = acquire(ctx, &ctx->pack_buf, &ctx->pack_bytes, want, &pack);
                if (st) return st;
                if (!ctx->static_mode) {
                    parts = ensure_for_speed(ctx, &ctx->pack_buf, &ctx->pack_bytes, want);
                    pack = ctx->pack_buf;
                }
            }
            if (parts && kept) use_images();
            e = parts ? launch_sweep_b16(a, pack, want, ctx->stream) : launch_sweep(a, ctx->stream);
        }
        if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "launch_sweep", e);
        ctx->static_used = mark_used; // the next column group reuses the image region (same stream: ordered)
    }
    if (after_sweep) (void)hipEventRecord(after_sweep, ctx->stream);
    if (merged) {
        hipError_t e = launch_merge(part_is_64 ? nullptr : part, part_is_64 ? reinterpret_cast<double *>(part) : nullptr,
                                    chunks, nF * t, 1, out64 != nullptr ? nullptr : out, out64, 1, nF * t, ctx->stream);
        if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "launch_merge", e);
    }
    return KNM_OK;
}

static void mark(knm_ctx *ctx, int i)
{
    if (ctx->timing) {
        (void)hipEventRecord(ctx->ev[i], ctx->stream);
        ctx->ev_used[i] = true;
    }
}

static void begin_timing(knm_ctx *ctx)
{
    for (int i = 0; i < 5; ++i) ctx->ev_used[i] = false;
    mark(ctx, 0);
}

int do_knm_v(knm_ctx *ctx, const float *X, int64_t n, int d, int64_t ldx, const float *C, int64_t M,
             int64_t ldc, float sigma, const float *V, int t, float *W)
{
    TraceRange range("knm row sweep W = K V");
    return sweep(ctx, X, n, ldx, C, M, ldc, d, sigma, V, nullptr, t, W, nullptr, nullptr, false);
}

int do_knm_t_w(knm_ctx *ctx, const float *X, int64_t n, int d, int64_t ldx, const float *C, int64_t M,
               int64_t ldc, float sigma, const float *Wv, const float *wgt, int t, float *U, double *U64)
{
    hipEvent_t ev = nullptr;
    if (ctx->timing) {
        ev = ctx->ev[2];
        ctx->ev_used[2] = true;
    }
    TraceRange range("knm column sweep U = K^T W");
    return sweep(ctx, C, M, ldc, X, n, ldx, d, sigma, Wv, wgt, t, U64 != nullptr ? nullptr : U, U64, ev, true);
}

} // namespace knm

using namespace knm;

extern "C" {

int knm_create(knm_ctx **out, int device, void *hip_stream)
{
    if (!out) return KNM_INVALID_ARG;
    *out = nullptr;
    int count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess || device < 0 || device >= count) return KNM_INVALID_ARG;
    if (hipSetDevice(device) != hipSuccess) return KNM_HIP_ERROR;
    knm_ctx *ctx = new (std::nothrow) knm_ctx();
    if (!ctx) return KNM_ALLOC;
    ctx->device = device;
    ctx->stream = static_cast<hipStream_t>(hip_stream);
    {
        // this device's copy of the static scratch array (the device is current)
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) {
            (void)hipGetLastError();
            delete ctx;
            return KNM_HIP_ERROR;
        }
        ctx->static_ws = static_cast<unsigned char *>(ptr);
    }
    for (int i = 0; i < 5; ++i) {
        if (hipEventCreate(&ctx->ev[i]) != hipSuccess) {
            (void)knm_destroy(ctx);
            return KNM_HIP_ERROR;
        }
    }
    {
        // the word the split-fp16 engines count clamped operands in (allocated here so that the
        // products themselves never allocate for it)
        void *w = nullptr;
        if (hipMalloc(&w, 256) != hipSuccess || hipMemset(w, 0, 256) != hipSuccess) {
            (void)hipGetLastError();
            if (w) (void)hipFree(w);
            (void)knm_destroy(ctx);
            return KNM_ALLOC;
        }
        ctx->range_count = static_cast<unsigned int *>(w);
    }
    *out = ctx;
    return KNM_OK;
}

int knm_destroy(knm_ctx *ctx)
{
    if (!ctx) return KNM_INVALID_ARG;
    (void)hipStreamSynchronize(ctx->stream);
    if (ctx->w_buf) (void)hipFree(ctx->w_buf);
    if (ctx->part_buf) (void)hipFree(ctx->part_buf);
    if (ctx->pack_buf) (void)hipFree(ctx->pack_buf);
    if (ctx->vimg_buf) (void)hipFree(ctx->vimg_buf);
    if (ctx->mu_buf) (void)hipFree(ctx->mu_buf);
    if (ctx->range_count) (void)hipFree(ctx->range_count);
    for (auto &b : ctx->pool) (void)hipFree(b.p);
    for (int i = 0; i < 5; ++i)
        if (ctx->ev[i]) (void)hipEventDestroy(ctx->ev[i]);
    extern void knm_solver_release(knm_ctx *);
    knm_solver_release(ctx);
    delete ctx;
    return KNM_OK;
}

const char *knm_strerror(int status)
{
    switch (status) {
    case KNM_OK: return "ok";
    case KNM_INVALID_ARG: return "invalid argument";
    case KNM_UNSUPPORTED: return "shape not supported by the compiled kernels";
    case KNM_ALLOC: return "device workspace allocation failed";
    case KNM_HIP_ERROR: return "HIP runtime or library error";
    case KNM_NOT_PD: return "matrix not positive definite in Cholesky factorisation";
    default: return "unknown status";
    }
}

const char *knm_last_error(const knm_ctx *ctx) { return ctx ? ctx->last_error.c_str() : ""; }

int knm_max_d(void) { return 65536; }
int knm_max_t(void) { return 1024; }

size_t knm_workspace_bytes(int64_t n, int64_t M, int d, int t)
{
    if (n <= 0 || M <= 0 || d <= 0 || t <= 0) return 0;
    int64_t len = 0;
    const size_t bytes = sizeof(float) * (size_t)n * t; // W
    // the largest needs over the arithmetic modes and kernel functions (they may cut the stream
    // differently): chunk partials, and the packed operands of the split-fp16 modes
    size_t part = 0, pack = 0, vimg = 0, keep = 0;
    const int64_t sets[2] = {n, M};
    if (direct_pays(n, M, d, t, true, KNM_CROSS_F16X3) || direct_pays(n, M, d, t, true, KNM_CROSS_F32)) part = sizeof(double) * (size_t)direct_chunks(n, M, t) * n * t; // of a small K V
    for (int mode = 0; mode < 4; ++mode) {
        const int cross = mode & 1, kind = mode >> 1;
        const int64_t c1 = choose_chunks(n, M, d, t, cross, kind, &len);
        const int64_t l1 = len;
        const int64_t c2 = choose_chunks(M, n, d, t, cross, kind, &len);
        const int64_t l2 = len;
        const size_t p1 = c1 > 1 ? sizeof(float) * (size_t)c1 * n * t : 0;
        const size_t p2 = c2 > 1 ? sizeof(float) * (size_t)c2 * M * t : 0;
        if (p1 > part) part = p1;
        if (p2 > part) part = p2;
        if (const int64_t rows = product_keep_rows(n, M, d, t, cross, kind); rows > 0 && t > kept_rows_max_t()) {
            const size_t k = ManyPlan(n, rows, M, d, t).bytes;
            if (k > keep) keep = k;
        } else if (rows > 0) {
            // a slab of values, the partials and running sums of the sums over it, weighted rows (256 bytes of rounding each)
            const size_t k = kept_bytes(rows, M) + p2 + sizeof(double) * 4 * (size_t)M * t + sizeof(float) * (size_t)(rows + M) * t + 1024;
            if (k > keep) keep = k;
            for (int64_t nr : {rows, n % rows}) { // the last slab is cut into chunks by itself
                const int64_t c3 = nr > 0 ? choose_chunks(nr, M, d, t, cross, kind, &len) : 0;
                if (c3 > 1 && sizeof(float) * (size_t)c3 * nr * t > part) part = sizeof(float) * (size_t)c3 * nr * t;
            }
        }
        if (packs_images(n, M, d, t, cross, kind)) {
            const size_t k1 = pack_bytes_wanted(n, d, t, cross, kind, 0, c1, l1);
            const size_t k2 = pack_bytes_wanted(M, d, t, cross, kind, 0, c2, l2);
            if (k1 > pack) pack = k1;
            if (k2 > pack) pack = k2;
        }
        if (cross == KNM_CROSS_F16X3) {
            const size_t both = product_image_bytes(sets, d, t, kind, 0);
            if (both > 0 && both + gemm_f16_head_bytes() > pack) pack = both + gemm_f16_head_bytes();
            if (use_gemm_engine(d, t, cross, kind)) {
                // packed vector image of the widest launch (matrix-core reduction), for either sweep
                const int wide = t < gemm_f16_max_t(kind) ? t : gemm_f16_max_t(kind);
                const size_t v1 = gemm_f16_vector_image_bytes(d, wide, c1 * l1), v2 = gemm_f16_vector_image_bytes(d, wide, c2 * l2);
                if (v1 <= kVectorImageCap && v1 > vimg) vimg = v1;
                if (v2 <= kVectorImageCap && v2 > vimg) vimg = v2;
            }
        }
    }
    return bytes + part + pack + vimg + keep + mu_bytes_wanted(kMeanSample, d);
}

size_t knm_workspace_held(const knm_ctx *ctx)
{
    if (!ctx) return 0;
    return ctx->w_bytes + ctx->part_bytes + ctx->pack_bytes + ctx->vimg_bytes + ctx->mu_bytes + ctx->pool_idle + (ctx->slab ? ctx->slab_bytes : 0);
}

int knm_release_workspace(knm_ctx *ctx)
{
    if (!ctx) return KNM_INVALID_ARG;
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipSetDevice");
    hipError_t e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "knm_release_workspace", e);
    for (auto held : {std::make_pair(&ctx->w_buf, &ctx->w_bytes), std::make_pair(&ctx->part_buf, &ctx->part_bytes),
                      std::make_pair(&ctx->pack_buf, &ctx->pack_bytes), std::make_pair(&ctx->vimg_buf, &ctx->vimg_bytes),
                      std::make_pair(&ctx->mu_buf, &ctx->mu_bytes)}) {
        const hipError_t freed = *held.first ? hipFree(*held.first) : hipSuccess;
        if (e == hipSuccess) e = freed;
        *held.first = nullptr;
        *held.second = 0;
    }
    drop_slab(ctx);
    const std::lock_guard<std::mutex> lock(ctx->pool_lock);
    free_idle_locked(ctx);
    return e == hipSuccess ? KNM_OK : fail(ctx, KNM_HIP_ERROR, "knm_release_workspace", e);
}

static int check_common(knm_ctx *ctx, const void *X, int64_t n, int d, int64_t ldx, const void *C, int64_t M,
                        int64_t ldc, float sigma, int t)
{
    if (!ctx) return KNM_INVALID_ARG;
    if (bad_geom(X, n, d, ldx, C, M, ldc, sigma, t)) return fail(ctx, KNM_INVALID_ARG, "bad shape or pointer");
    if (d > knm_max_d() || t > knm_max_t()) return fail(ctx, KNM_UNSUPPORTED, "d or t above compiled maximum");
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipSetDevice");
    return KNM_OK;
}

static int small_knm_v(knm_ctx *ctx, const float *X, int64_t n, int d, int64_t ldx, const float *C, int64_t M, int64_t ldc, float sigma,
                       const float *V, int t, float *W)
{
    TraceRange range("knm small row sweep W = K V");
    const int chunks = direct_chunks(n, M, t);
    double *part = nullptr;
    if (chunks > 1) {
        int st = ensure(ctx, &ctx->part_buf, &ctx->part_bytes, sizeof(double) * (size_t)chunks * n * t);
        if (st) return st;
        part = reinterpret_cast<double *>(ctx->part_buf);
    }
    hipError_t e = launch_direct(X, n, ldx, C, M, ldc, d, engine_sigma(sigma, ctx->kernel_kind), ctx->kernel_kind, V, t, W, part,
                                 ctx->cross_term == KNM_CROSS_F16X3 ? ctx->range_count : nullptr, 1.0f / (2.0f * sigma * sigma), ctx->stream);
    if (e == hipSuccess && part != nullptr) e = launch_merge(nullptr, part, chunks, n * t, 1, W, nullptr, 1, n * t, ctx->stream);
    return e == hipSuccess ? KNM_OK : fail(ctx, KNM_HIP_ERROR, "launch_direct", e);
}

int knm_v(knm_ctx *ctx, const float *X, int64_t n, int d, int64_t ldx, const float *C, int64_t M, int64_t ldc,
          float sigma, const float *V, int t, float *W)
{
    int st = check_common(ctx, X, n, d, ldx, C, M, ldc, sigma, t);
    if (st) return st;
    if (!V || !W) return fail(ctx, KNM_INVALID_ARG, "null vector");
    begin_timing(ctx);
    if (direct_takes(sigma) && direct_pays(n, M, d, t, direct_wide(C, ldc, d), ctx->cross_term)) st = small_knm_v(ctx, X, n, d, ldx, C, M, ldc, sigma, V, t, W);
    else st = do_knm_v(ctx, X, n, d, ldx, C, M, ldc, sigma, V, t, W);
    mark(ctx, 1);
    mark(ctx, 4);
    return st;
}

// out[i, c] = w[i] x[i, c] for count = rows x t entries
__global__ void weigh_rows_kernel(const float *__restrict__ x, const float *__restrict__ w, int64_t count, int t, float *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) out[i] = x[i] * w[i / t];
}

// The product with the kernel values of a slab of rows kept from its row sweep to its share of the sums over the columns: every value
// is formed once.  *done = false: no room.
static int prod_kept(knm_ctx *ctx, const float *X, int64_t n, int d, int64_t ldx, const float *C, int64_t M, int64_t ldc, float sigma,
                     const float *dw, const float *V, int t, float *W, float *U, int64_t rows, bool *done)
{
    *done = false;
    KeptRowsArgs k{};
    const int64_t chunks = choose_chunks(M, n, d, t, ctx->cross_term, ctx->kernel_kind, &k.chunk_len);
    if (chunks > 65535) return KNM_OK;
    // values, chunk partials, running sums, weighted rows
    const size_t pieces[4] = {kept_bytes(rows, M), sizeof(float) * (size_t)chunks * M * t, sizeof(double) * 4 * (size_t)M * t,
                              dw != nullptr ? sizeof(float) * (size_t)rows * t : 0};
    size_t at[4], bytes = 0;
    for (int i = 0; i < 4; ++i) {
        at[i] = bytes;
        bytes += (pieces[i] + 255) & ~(size_t)255;
    }
    const SlabUse slab(ctx, bytes);
    if (slab.p == nullptr) return KNM_OK;
    auto piece = [&](int i) { return static_cast<void *>(static_cast<char *>(slab.p) + at[i]); };
    SweepShare share(ctx, X, n, ldx, C, M, ldc, d, sigma, t, false); // (the shift is that of the whole pair, for all slabs)
    share.n[0] = rows;
    share.slab = static_cast<float *>(piece(0));
    const ShareScope scope(share);
    k.values = share.slab;
    k.n = n;
    k.nS = M;
    k.t = t;
    k.part = static_cast<float *>(piece(1));
    double *s_in = static_cast<double *>(piece(2)), *s_out = s_in + 2 * (size_t)M * t;
    for (k.row0 = 0; k.row0 < n; k.row0 += rows, std::swap(s_in, s_out)) {
        k.rows = n - k.row0 < rows ? n - k.row0 : rows;
        share.P[0] = X + k.row0 * ldx;
        share.n[0] = k.rows;
        share.ready[0] = 0;
        float *Wb = W + k.row0 * t;
        const int st = do_knm_v(ctx, share.P[0], k.rows, d, ldx, C, M, ldc, sigma, V, t, Wb);
        if (st == KNM_ALLOC) return KNM_OK; // without the slab there may be room
        if (st) return st;
        if (k.row0 + rows >= n) mark(ctx, 1);
        TraceRange range("knm column sums of a slab");
        k.vec = Wb;
        if (dw != nullptr) {
            const int64_t count = k.rows * t;
            float *const weighted = static_cast<float *>(piece(3));
            k.vec = weighted;
            hipLaunchKernelGGL(weigh_rows_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, ctx->stream, Wb, dw + k.row0, count, t,
                               weighted);
        }
        k.state_in = s_in;
        k.state_out = s_out;
        const hipError_t e = launch_kept_rows(k, ctx->stream);
        if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "launch_kept_rows", e);
    }
    mark(ctx, 2);
    const hipError_t e = launch_merge(k.part, nullptr, chunks, M * t, 1, U, nullptr, 1, M * t, ctx->stream);
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "launch_merge", e);
    mark(ctx, 3);
    mark(ctx, 4);
    *done = true;
    return KNM_OK;
}

// u64[j] (+)= the partials' sum in a fixed order; the last slab's goes out in fp32
__global__ __launch_bounds__(256) void add_partials_kernel(const float *__restrict__ part, int64_t n_chunks, int64_t count, int first, int last,
                                                           double *__restrict__ u64, float *__restrict__ out)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= count) return;
    double s = first ? 0.0 : u64[j];
    int64_t c = 0;
    for (; c + 4 <= n_chunks; c += 4) {
        const float p0 = part[c * count + j], p1 = part[(c + 1) * count + j], p2 = part[(c + 2) * count + j], p3 = part[(c + 3) * count + j];
        s += ((double)p0 + (double)p1) + ((double)p2 + (double)p3);
    }
    for (; c < n_chunks; ++c) s += (double)part[c * count + j];
    if (last) out[j] = (float)s;
    else u64[j] = s;
}

// The product with many columns from kernel values that are formed once: slab by slab of rows, the values, W from them and the slab's share
// of U.  *done = false: no room.
static int prod_kept_many(knm_ctx *ctx, const float *X, int64_t n, int d, int64_t ldx, const float *C, int64_t M, int64_t ldc, float sigma,
                          const float *dw, const float *V, int t, float *W, float *U, int64_t rows, bool *done)
{
    *done = false;
    const ManyPlan plan(n, rows, M, d, t);
    const SlabUse slab(ctx, plan.bytes);
    if (slab.p == nullptr) return KNM_OK;
    auto piece = [&](int i) { return static_cast<void *>(static_cast<char *>(slab.p) + plan.at[i]); };
    float *const values = static_cast<float *>(piece(0)), *const part_w = static_cast<float *>(piece(1)), *const part_u = static_cast<float *>(piece(2));
    double *const u64 = static_cast<double *>(piece(3));
    uint32_t *const scales[2] = {static_cast<uint32_t *>(piece(6)), static_cast<uint32_t *>(piece(6)) + gemm_f16_head_bytes() / sizeof(uint32_t)};
    SweepShare share(ctx, X, n, ldx, C, M, ldc, d, sigma, t, false); // (the shift is that of the whole pair, for all slabs)
    share.n[0] = rows;
    const ShareScope scope(share);
    float *mu = nullptr;
    int st = acquire(ctx, &ctx->mu_buf, &ctx->mu_bytes, mu_bytes_wanted(share.shift_n, d), &mu);
    if (!st) st = column_shift(ctx, share.shift_P, share.shift_n, share.shift_ld, d, sigma, mu);
    if (st) return st;
    ctx->mu_owner = &share;
    st = share_images(ctx, &share);
    if (st == KNM_ALLOC || (!st && share.img[0] == nullptr)) return KNM_OK;
    if (st) return st;
    auto failed = [&](hipError_t e, const char *what) { return e == hipSuccess ? KNM_OK : fail(ctx, KNM_HIP_ERROR, what, e); };
    auto image = [&](const float *vec, const float *wgt, int64_t count, int columns, int which) {
        return failed(launch_vector_image(vec, t, wgt, count, (count + 127) / 128 * 128, columns, scales[which], piece(4 + which), ctx->stream),
                      "launch_vector_image");
    };
    KeptManyArgs k{};
    k.values = values;
    k.nS = M;
    k.ldo = t;
    for (int64_t row0 = 0; row0 < n; row0 += rows) {
        k.nF = n - row0 < rows ? n - row0 : rows;
        share.P[0] = X + row0 * ldx;
        share.n[0] = k.nF;
        share.ready[0] = 0;
        float *const Wb = W + row0 * t;
        {
            TraceRange range("knm kernel values of a slab");
            st = form_values(ctx, &share, 0, 1, mu, values);
            if (st) return st;
        }
        TraceRange range("knm sums over a slab's kernel values");
        for (int side = 0; side < 2; ++side) { // W of the slab's rows, then their share of U
            if (side == 1 && row0 + rows >= n) mark(ctx, 1);
            const int64_t n_in = side == 0 ? M : k.nF, n_out = side == 0 ? k.nF : M;
            k.over_stream = side == 0;
            k.chunk_len = side == 0 ? plan.row_chunk : plan.col_chunk;
            k.part_stride = n_out * t;
            for (int c = 0; c < t; c += plan.group) {
                k.t = t - c < plan.group ? t - c : plan.group;
                if (side == 1) st = image(Wb + c, dw != nullptr ? dw + row0 : nullptr, k.nF, k.t, 1);
                else if (row0 == 0 || t > plan.group) st = image(V + c, nullptr, M, k.t, 0);
                if (st) return st;
                k.vimg = piece(4 + side);
                k.colmax = scales[side];
                k.part = (side == 0 ? part_w : part_u) + c;
                st = failed(launch_kept_many(k, ctx->stream), "launch_kept_many");
                if (st) return st;
            }
            const int64_t chunks = (n_in + k.chunk_len - 1) / k.chunk_len, count = n_out * t;
            if (side == 0) st = failed(launch_merge(part_w, nullptr, chunks, count, 1, Wb, nullptr, 1, count, ctx->stream), "launch_merge");
            else {
                if (row0 + rows >= n) mark(ctx, 2);
                hipLaunchKernelGGL(add_partials_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, ctx->stream, part_u, chunks, count,
                                   row0 == 0 ? 1 : 0, row0 + rows >= n ? 1 : 0, u64, U);
                st = failed(hipGetLastError(), "add_partials_kernel");
            }
            if (st) return st;
        }
    }
    mark(ctx, 3);
    mark(ctx, 4);
    *done = true;
    return KNM_OK;
}

static int prod_impl(knm_ctx *ctx, const float *X, int64_t n, int d, int64_t ldx, const float *C, int64_t M,
                     int64_t ldc, float sigma, const float *dw, const float *V, int t, float *W_or_null, float *U)
{
    int st = check_common(ctx, X, n, d, ldx, C, M, ldc, sigma, t);
    if (st) return st;
    if (!V || !U) return fail(ctx, KNM_INVALID_ARG, "null vector");
    float *W = W_or_null;
    if (!W) {
        st = ensure(ctx, &ctx->w_buf, &ctx->w_bytes, sizeof(float) * (size_t)n * t);
        if (st) return st;
        W = ctx->w_buf;
    }
    begin_timing(ctx);
    const int64_t keep_rows = ctx->static_mode ? 0 : product_keep_rows(n, M, d, t, ctx->cross_term, ctx->kernel_kind);
    if (keep_rows > 0) {
        bool done = false;
        st = (t > kept_rows_max_t() ? prod_kept_many : prod_kept)(ctx, X, n, d, ldx, C, M, ldc, sigma, dw, V, t, W, U, keep_rows, &done);
        if (st || done) return st;
        begin_timing(ctx);
    }
    SweepShare share(ctx, X, n, ldx, C, M, ldc, d, sigma, t, false);
    const ShareScope scope(share);
    st = do_knm_v(ctx, X, n, d, ldx, C, M, ldc, sigma, V, t, W);
    if (st) return st;
    mark(ctx, 1);
    st = do_knm_t_w(ctx, X, n, d, ldx, C, M, ldc, sigma, W, dw, t, U);
    if (st) return st;
    mark(ctx, 3);
    mark(ctx, 4);
    return KNM_OK;
}

int knm_prod(knm_ctx *ctx, const float *X, int64_t n, int d, int64_t ldx, const float *C, int64_t M, int64_t ldc,
             float sigma, const float *V, int t, float *W_or_null, float *U)
{
    return prod_impl(ctx, X, n, d, ldx, C, M, ldc, sigma, nullptr, V, t, W_or_null, U);
}

size_t knm_static_scratch_bytes(void) { return kStaticScratchBytes; }

int knm_prod_static(knm_ctx *ctx, const float *X, int64_t n, int d, int64_t ldx, const float *C, int64_t M, int64_t ldc,
                    float sigma, const float *V, int t, float *W, float *U)
{
    if (ctx && !W) return fail(ctx, KNM_INVALID_ARG, "the allocation-free product needs the caller's W");
    if (!ctx) return KNM_INVALID_ARG;
    ctx->static_mode = true;
    const int st = prod_impl(ctx, X, n, d, ldx, C, M, ldc, sigma, nullptr, V, t, W, U);
    ctx->static_mode = false;
    return st;
}

int knm_prod_weighted(knm_ctx *ctx, const float *X, int64_t n, int d, int64_t ldx, const float *C, int64_t M,
                      int64_t ldc, float sigma, const float *dw, const float *V, int t, float *U)
{
    if (ctx && !dw) return fail(ctx, KNM_INVALID_ARG, "null weights");
    return prod_impl(ctx, X, n, d, ldx, C, M, ldc, sigma, dw, V, t, nullptr, U);
}

int knm_t_y(knm_ctx *ctx, const float *X, int64_t n, int d, int64_t ldx, const float *C, int64_t M, int64_t ldc,
            float sigma, const float *Y, int t, float *R)
{
    int st = check_common(ctx, X, n, d, ldx, C, M, ldc, sigma, t);
    if (st) return st;
    if (!Y || !R) return fail(ctx, KNM_INVALID_ARG, "null vector");
    begin_timing(ctx);
    mark(ctx, 1);
    st = do_knm_t_w(ctx, X, n, d, ldx, C, M, ldc, sigma, Y, nullptr, t, R);
    if (st) return st;
    mark(ctx, 3);
    mark(ctx, 4);
    return KNM_OK;
}

int knm_range_exceeded(knm_ctx *ctx, int64_t *count_host, int reset)
{
    if (!ctx) return KNM_INVALID_ARG;
    if (!count_host) return fail(ctx, KNM_INVALID_ARG, "null count");
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipSetDevice");
    unsigned int c = 0;
    hipError_t e = hipMemcpyAsync(&c, ctx->range_count, sizeof(c), hipMemcpyDeviceToHost, ctx->stream);
    if (e == hipSuccess && reset) e = hipMemsetAsync(ctx->range_count, 0, sizeof(c), ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "knm_range_exceeded", e);
    *count_host = (int64_t)c;
    return KNM_OK;
}

int knm_set_cross_term(knm_ctx *ctx, int mode)
{
    if (!ctx) return KNM_INVALID_ARG;
    if (mode != KNM_CROSS_F32 && mode != KNM_CROSS_F16X3) return fail(ctx, KNM_INVALID_ARG, "unknown cross-term mode");
    ctx->cross_term = mode;
    return KNM_OK;
}

int knm_get_cross_term(const knm_ctx *ctx) { return ctx ? ctx->cross_term : KNM_INVALID_ARG; }

int knm_set_kernel(knm_ctx *ctx, int kind)
{
    if (!ctx) return KNM_INVALID_ARG;
    if (kind < KNM_KERNEL_GAUSSIAN || kind > KNM_KERNEL_MATERN52) return fail(ctx, KNM_INVALID_ARG, "unknown kernel");
    ctx->kernel_kind = kind;
    return KNM_OK;
}

int knm_set_sparse_head_limit(knm_ctx *ctx, int max_features)
{
    if (!ctx) return KNM_INVALID_ARG;
    if (max_features < 0) return fail(ctx, KNM_INVALID_ARG, "negative head limit");
    ctx->sparse_head_max = max_features > 128 ? 128 : max_features;
    return KNM_OK;
}

int knm_set_pack_limit(knm_ctx *ctx, size_t bytes)
{
    if (!ctx) return KNM_INVALID_ARG;
    ctx->pack_limit = bytes;
    return KNM_OK;
}

int knm_set_timing(knm_ctx *ctx, int enabled)
{
    if (!ctx) return KNM_INVALID_ARG;
    ctx->timing = enabled != 0;
    for (int i = 0; i < 5; ++i) ctx->ev_used[i] = false;
    return KNM_OK;
}

int knm_get_timing(knm_ctx *ctx, float *ms)
{
    if (!ctx || !ms) return KNM_INVALID_ARG;
    for (int i = 0; i < 4; ++i) ms[i] = 0.0f;
    if (!ctx->ev_used[0] || !ctx->ev_used[4]) return fail(ctx, KNM_INVALID_ARG, "no timed call recorded");
    hipError_t e = hipEventSynchronize(ctx->ev[4]);
    if (e != hipSuccess) return fail(ctx, KNM_HIP_ERROR, "hipEventSynchronize", e);
    // events: 0 start, 1 after row sweep, 2 after column sweep kernels, 3 after merge, 4 end
    auto span = [&](int a, int b, float *dst) {
        if (ctx->ev_used[a] && ctx->ev_used[b]) (void)hipEventElapsedTime(dst, ctx->ev[a], ctx->ev[b]);
    };
    span(0, 1, &ms[0]);
    span(1, 2, &ms[1]);
    span(2, 3, &ms[2]);
    span(0, 4, &ms[3]);
    return KNM_OK;
}

} // extern "C"
