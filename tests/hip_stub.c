/* The HIP entry points that libgp.so imports, on host memory and without a
 * device: kernels do nothing, copies copy. Host code (allocation failures, what
 * is allocated and launched) runs against it in a process without a GPU. */
#include <errno.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef int err;
enum { OK = 0, OOM = 2, NOT_SUPPORTED = 801 };

static err last;              /* what hipGetLastError hands out, then clears */
static int64_t host_allocs;   /* successful hipHostMalloc calls */
static int64_t fail_host;     /* hipHostMalloc calls still to fail */
static int64_t pool_idle;     /* bytes freed to pools and not trimmed */
static int64_t device_limit;  /* hipMalloc and hipMallocAsync fail above limit - pool_idle bytes (0: never) */
static int64_t trims;

int64_t stub_host_allocs(void) { return host_allocs; }
int64_t stub_pool_idle(void) { return pool_idle; }
int64_t stub_trims(void) { return trims; }
void stub_fail_host(int64_t n) { fail_host = n; }
void stub_device_limit(int64_t bytes) { device_limit = bytes; }

static err fail(err e) { return last = e; }

/* device blocks carry their size and whether a pool owns them */
struct head {
    int64_t bytes;
    int64_t pooled;
    char pad[240];
};
static err device_alloc(void** p, size_t n, int pooled) {
    if (device_limit && (int64_t)n > device_limit - pool_idle) return fail(OOM);
    struct head* h = aligned_alloc(256, (sizeof(struct head) + n + 255) / 256 * 256);
    if (!h) return fail(OOM);
    h->bytes = (int64_t)n;
    h->pooled = pooled;
    memset(h + 1, 0, n);
    *p = h + 1;
    return OK;
}
static err device_free(void* p) {
    if (p) {
        struct head* h = (struct head*)p - 1;
        if (h->pooled) pool_idle += h->bytes;
        free(h);
    }
    return OK;
}

err hipMalloc(void** p, size_t n) { return device_alloc(p, n, 0); }
err hipFree(void* p) { return device_free(p); }
err hipMallocAsync(void** p, size_t n, void* s) { return device_alloc(p, n, 0); }
err hipMallocFromPoolAsync(void** p, size_t n, void* pool, void* s) {
    if ((int64_t)n <= pool_idle) {  /* served by what the pool holds */
        pool_idle -= (int64_t)n;
        const int64_t limit = device_limit;
        device_limit = 0;
        const err e = device_alloc(p, n, 1);
        device_limit = limit;
        return e;
    }
    return device_alloc(p, n, 1);
}
err hipFreeAsync(void* p, void* s) { return device_free(p); }
err hipMemPoolCreate(void** pool, const void* props) { *pool = malloc(8); return OK; }
err hipMemPoolDestroy(void* pool) { free(pool); return OK; }
err hipMemPoolSetAttribute(void* pool, int a, void* v) { return OK; }
err hipMemPoolTrimTo(void* pool, size_t keep) { ++trims; pool_idle = 0; return OK; }
err hipHostMalloc(void** p, size_t n, unsigned f) {
    if (fail_host > 0) {
        --fail_host;
        return fail(OOM);
    }
    ++host_allocs;
    *p = calloc(1, n);
    return OK;
}
err hipHostFree(void* p) { free(p); return OK; }
err hipMemcpy(void* d, const void* s, size_t n, int k) { memcpy(d, s, n); return OK; }
err hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { memcpy(d, s, n); return OK; }
err hipMemsetAsync(void* d, int v, size_t n, void* st) { memset(d, v, n); return OK; }

err hipGetLastError(void) {
    const err e = last;
    last = OK;
    return e;
}
err hipGetDevice(int* d) { *d = 0; return OK; }
err hipSetDevice(int d) { return OK; }
err hipGetStreamDeviceId(void* s) { return 0; }
err hipDeviceSynchronize(void) { return OK; }
err hipDeviceGetAttribute(int* v, int a, int d) { *v = 256; return OK; }
err hipGetDevicePropertiesR0600(char* p, int d) {
    strcpy(p + 1160, "gfx950"); /* gcnArchName: the library's sorts pick their tuning by it */
    return OK;
}
err hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int b, size_t s) { *n = 8; return OK; }
err hipGetSymbolAddress(void** p, const void* sym) { return fail(NOT_SUPPORTED); }

static int token;
err hipStreamCreateWithFlags(void** s, unsigned f) { *s = &token; return OK; }
err hipStreamDestroy(void* s) { return OK; }
err hipStreamSynchronize(void* s) { return OK; }
err hipStreamIsCapturing(void* s, int* st) { *st = 0; return OK; }
err hipStreamBeginCapture(void* s, int m) { return OK; }
err hipStreamEndCapture(void* s, void** g) { *g = &token; return OK; }
err hipEventCreate(void** e) { *e = &token; return OK; }
err hipEventCreateWithFlags(void** e, unsigned f) { *e = &token; return OK; }
err hipEventDestroy(void* e) { return OK; }
err hipEventRecord(void* e, void* s) { return OK; }
err hipEventQuery(void* e) { return OK; }
err hipEventSynchronize(void* e) { return OK; }
err hipEventElapsedTime(float* ms, void* a, void* b) { *ms = 1; return OK; }
err hipGraphInstantiate(void** x, void* g, void** n, char* l, size_t b) { *x = &token; return OK; }
err hipGraphLaunch(void* x, void* s) { return OK; }
err hipGraphDestroy(void* g) { return OK; }
err hipGraphExecDestroy(void* x) { return OK; }

struct dim3 {
    uint32_t x, y, z;
};
err hipLaunchKernel(const void* f, struct dim3 g, struct dim3 b, void** a, size_t l, void* s) { return OK; }
err __hipPushCallConfiguration(struct dim3 g, struct dim3 b, size_t l, void* s) { return OK; }
err __hipPopCallConfiguration(struct dim3* g, struct dim3* b, size_t* l, void** s) {
    *l = 0;
    *s = 0;
    return OK;
}
void** __hipRegisterFatBinary(const void* d) {
    static void* h;
    return &h;
}
void __hipRegisterFunction(void** m, const void* h, char* d, const char* n, unsigned t, void* a, void* b, void* c,
                           void* e, int* w) {}
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t n, int c, int g) {}
void __hipUnregisterFatBinary(void** m) {}
