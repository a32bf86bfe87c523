/* A stand-in for the HIP runtime, for tests of librcx's host code without a
 * GPU (tests/host_runtime.py): device memory is lazily mapped host memory,
 * kernels do nothing, and every launch is logged with its name and grid. A
 * launch of 2^32 work items or more along an axis, or a grid past 65535 in y
 * or z, fails as the runtime fails it. fake_fail_malloc(n, m) makes the
 * allocations n .. n + m - 1 from now on (0 = the next) fail for want of memory. */
#define _GNU_SOURCE
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

enum { kOk = 0, kInvalidValue = 1, kOutOfMemory = 2, kInvalidConfiguration = 9 };
typedef struct { uint32_t x, y, z; } dim3_t;

static struct { void* p; size_t n; } mem[65536];
static int n_mem, fail_at = -1, fail_count, last_error;
static struct { const void* fn; char name[512]; } fns[1024];
static int n_fns;
static char* log_text;
static size_t log_len, log_cap;
static size_t live, sizes[256];
static int n_sizes;

static int set(int e)
{
    if (e != kOk) last_error = e;
    return e;
}

void fake_fail_malloc(int n, int m) { fail_at = n; fail_count = m; }
size_t fake_live_bytes(void) { return live; }
/* sizes of the allocations asked for since the last call */
int fake_sizes(size_t* out) { int n = n_sizes; memcpy(out, sizes, sizeof(size_t) * (size_t)n); n_sizes = 0; return n; }
const char* fake_log(void) { return log_text ? log_text : ""; }
void fake_log_clear(void) { log_len = 0; if (log_text) log_text[0] = 0; }

int hipMalloc(void** p, size_t n)
{
    *p = NULL;
    if (n_sizes < 256) sizes[n_sizes++] = n;
    if (fail_count > 0 && fail_at-- <= 0) {
        --fail_count;
        return set(kOutOfMemory);
    }
    if (n == 0) return kOk;
    void* q = mmap(NULL, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (q == MAP_FAILED || n_mem == 65536) return set(kOutOfMemory);
    mem[n_mem].p = q;
    mem[n_mem++].n = n;
    live += n;
    *p = q;
    return kOk;
}
int hipFree(void* p)
{
    if (!p) return kOk;
    for (int i = 0; i < n_mem; ++i)
        if (mem[i].p == p) {
            munmap(p, mem[i].n);
            live -= mem[i].n;
            mem[i] = mem[--n_mem];
            return kOk;
        }
    return set(kInvalidValue);
}
int hipHostMalloc(void** p, size_t n, unsigned flags) { (void)flags; *p = calloc(1, n); return *p ? kOk : set(kOutOfMemory); }
int hipHostFree(void* p) { free(p); return kOk; }
int hipMemcpy(void* d, const void* s, size_t n, int kind) { (void)kind; memcpy(d, s, n); return kOk; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* st) { (void)st; return hipMemcpy(d, s, n, kind); }
int hipMemset(void* d, int v, size_t n) { memset(d, v, n); return kOk; }
int hipGetLastError(void) { int e = last_error; last_error = kOk; return e; }
const char* hipGetErrorName(int e) { return e == kOutOfMemory ? "hipErrorOutOfMemory" : "hipError"; }
const char* hipGetErrorString(int e) { return hipGetErrorName(e); }
/* every field 0 (the structure holds 1472 bytes) */
int hipGetDevicePropertiesR0600(void* prop, int d) { (void)d; memset(prop, 0, 1472); return kOk; }
int hipGetDevice(int* d) { *d = 0; return kOk; }
int hipDeviceSynchronize(void) { return kOk; }
int hipGetSymbolAddress(void** p, const void* sym)
{
    (void)sym;
    static void* scratch;
    if (!scratch) scratch = mmap(NULL, (size_t)64 << 20, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    *p = scratch;
    return kOk;
}
int hipStreamSynchronize(void* s) { (void)s; return kOk; }
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = malloc(1); return kOk; }
int hipStreamDestroy(void* s) { free(s); return kOk; }
int hipStreamWaitEvent(void* s, void* e, unsigned f) { (void)s; (void)e; (void)f; return kOk; }
int hipEventCreate(void** e) { *e = malloc(1); return kOk; }
int hipEventCreateWithFlags(void** e, unsigned f) { (void)f; return hipEventCreate(e); }
int hipEventDestroy(void* e) { free(e); return kOk; }
int hipEventRecord(void* e, void* s) { (void)e; (void)s; return kOk; }
int hipEventSynchronize(void* e) { (void)e; return kOk; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 1.0f; return kOk; }

void** __hipRegisterFatBinary(const void* d) { (void)d; static void* h; return &h; }
void __hipUnregisterFatBinary(void** h) { (void)h; }
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t s, int c, int g)
{
    (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g;
}
void __hipRegisterFunction(void** m, const void* fn, char* dev, const char* name, unsigned l, void* t, void* b, void* bd,
                           void* gd, int* w)
{
    (void)m; (void)dev; (void)l; (void)t; (void)b; (void)bd; (void)gd; (void)w;
    if (n_fns < 1024) {
        fns[n_fns].fn = fn;
        snprintf(fns[n_fns++].name, sizeof(fns[0].name), "%s", name);
    }
}
static struct { dim3_t g, b; size_t sh; void* st; } call;
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t sh, void* st)
{
    call.g = g; call.b = b; call.sh = sh; call.st = st;
    return kOk;
}
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* sh, void** st)
{
    *g = call.g; *b = call.b; *sh = call.sh; *st = call.st;
    return kOk;
}
int hipLaunchKernel(const void* fn, dim3_t g, dim3_t b, void** args, size_t sh, void* st)
{
    (void)args; (void)sh; (void)st;
    const char* name = "?";
    for (int i = 0; i < n_fns; ++i)
        if (fns[i].fn == fn) name = fns[i].name;
    if (log_cap - log_len < 1024) {
        log_cap = log_cap ? 2 * log_cap : 1 << 16;
        log_text = realloc(log_text, log_cap);
    }
    log_len += (size_t)snprintf(log_text + log_len, 1024, "%s %u %u %u %u\n", name, g.x, g.y, g.z, b.x);
    if (g.x == 0 || g.y == 0 || g.z == 0 || (uint64_t)g.x * b.x >> 32 || g.y > 65535 || g.z > 65535 || b.x > 1024)
        return set(kInvalidConfiguration);
    return kOk;
}
