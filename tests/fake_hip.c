/* A HIP runtime without a device, for tests of the library's host code: device memory is untouched address space with a
 * budget, kernels are not run, copies to the host read zeros.  Loaded before libknm with RTLD_GLOBAL its functions come first. */
#define _GNU_SOURCE
#include <stddef.h>
#include <stdint.h>
#include <string.h>
#include <sys/mman.h>

enum { kBlocks = 4096 };
static struct { void *p; size_t bytes; } blocks[kBlocks];
static size_t budget = (size_t)1 << 50, live, peak;
static long launches;
static int last_error;
static char device_symbol[256];

void fake_set_budget(size_t bytes) { budget = bytes; peak = live; }
size_t fake_live(void) { return live; }
size_t fake_peak(void) { return peak; }
long fake_launches(void) { return launches; }

int hipMalloc(void **out, size_t bytes)
{
    *out = NULL;
    if (bytes <= budget && live <= budget - bytes)
        for (int i = 0; i < kBlocks; ++i)
            if (blocks[i].p == NULL) {
                void *p = mmap(NULL, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
                if (p == MAP_FAILED) break;
                blocks[i].p = *out = p;
                blocks[i].bytes = bytes;
                live += bytes;
                if (live > peak) peak = live;
                return 0;
            }
    return last_error = 2; /* hipErrorOutOfMemory */
}
/* what a card of `total` bytes would say (0: no share of it matters) */
static size_t total;
void fake_set_total(size_t bytes) { total = bytes; }
int hipMemGetInfo(size_t *f, size_t *t) { *f = budget - live; *t = total; return 0; }
int hipFree(void *p)
{
    if (p == NULL) return 0;
    for (int i = 0; i < kBlocks; ++i)
        if (blocks[i].p == p) {
            munmap(p, blocks[i].bytes);
            live -= blocks[i].bytes;
            blocks[i].p = NULL;
            return 0;
        }
    return last_error = 1; /* hipErrorInvalidValue: freed twice, or not ours */
}
static int inside(const void *p, size_t bytes)
{
    const char *c = p;
    for (int i = 0; i < kBlocks; ++i)
        if (blocks[i].p != NULL && c >= (char *)blocks[i].p && c + bytes <= (char *)blocks[i].p + blocks[i].bytes) return 1;
    return 0;
}
/* kind 2: device to host, 3: within the device */
int hipMemcpyAsync(void *dst, const void *src, size_t bytes, int kind, void *stream)
{
    (void)stream;
    if (kind == 2) {
        if (!inside(src, bytes)) return last_error = 1;
        memset(dst, 0, bytes);
    }
    return 0;
}
int hipMemcpy(void *dst, const void *src, size_t bytes, int kind) { return hipMemcpyAsync(dst, src, bytes, kind, NULL); }
int hipMemset(void *p, int v, size_t bytes) { (void)v; return inside(p, bytes) ? 0 : (last_error = 1); }
int hipMemsetAsync(void *p, int v, size_t bytes, void *s) { (void)s; return hipMemset(p, v, bytes); }
int hipGetLastError(void) { const int e = last_error; last_error = 0; return e; }
const char *hipGetErrorString(int e) { return e == 2 ? "out of memory" : "error"; }
int hipGetDeviceCount(int *n) { *n = 1; return 0; }
int hipSetDevice(int d) { (void)d; return 0; }
int hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = device_symbol; return 0; }
int hipEventCreate(void **e) { *e = (void *)1; return 0; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; return hipEventCreate(e); }
int hipEventDestroy(void *e) { (void)e; return 0; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 0.0f; return 0; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = (void *)1; return 0; }
int hipStreamDestroy(void *s) { (void)s; return 0; }
int hipStreamSynchronize(void *s) { (void)s; return 0; }
int hipStreamWaitEvent(void *s, void *e, unsigned f) { (void)s; (void)e; (void)f; return 0; }
int hipFuncSetAttribute(const void *f, int a, int v) { (void)f; (void)a; (void)v; return 0; }
/* streams are not captured unless a test says so */
static int capturing;
void fake_set_capturing(int on) { capturing = on; }
int hipStreamIsCapturing(void *s, int *status) { (void)s; *status = capturing; return 0; }
int fake_inside(const void *p, size_t bytes) { return inside(p, bytes); }
int hipLaunchKernel(void) { ++launches; return 0; }
int __hipPushCallConfiguration(void) { return 0; }
int __hipPopCallConfiguration(void) { return 0; }
