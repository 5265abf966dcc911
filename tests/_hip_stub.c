/* A stand-in for the HIP runtime, for tests of the library's host code on a machine without a GPU: nothing runs, device
 * memory is host memory, and calls can be made to fail.  Loaded with global symbols before the library. */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
enum { OK = 0, OUT_OF_MEMORY = 2, LAUNCH_FAILURE = 719 };

static struct { const void *host; char name[256]; } kernels[4096];
static int num_kernels, last_error;
static struct { void *p; size_t bytes; int zeroed; } blocks[4096];
static int num_blocks;

/* what the test asks for and reads */
size_t stub_fail_alloc_bytes;                 /* allocations of this size fail */
size_t stub_fail_zero_bytes;                  /* and so does clearing of an allocation of this size, stub_fail_zero_times times */
int stub_fail_zero_times;
int stub_allocs_of_size, stub_device_syncs, stub_stream_syncs, stub_frees, stub_allocs;
size_t stub_alloc_bytes[4096];                /* what was asked for, in turn */
char stub_watch[64];                          /* a kernel's name: of its launches are noted */
int stub_watch_arg;                           /* the pointer that is this argument: */
int stub_watched, stub_watched_null, stub_watched_uncleared;

int stub_device;                              /* the current one; launches with more dynamic LDS than was allowed for the kernel there: */
int stub_lds_refused, stub_lds_calls;
static struct { const void *host; int device; size_t bytes; } lds[4096];
static size_t lds_allowed(const void *host) {
    size_t most = 65536;
    for (int i = 0; i < stub_lds_calls && i < 4096; ++i)
        if (lds[i].host == host && lds[i].device == stub_device && lds[i].bytes > most) most = lds[i].bytes;
    return most;
}

static int find(const void *p) {
    for (int i = 0; i < num_blocks; ++i)
        if (blocks[i].p && (char *)p >= (char *)blocks[i].p && (char *)p < (char *)blocks[i].p + blocks[i].bytes) return i;
    return -1;
}
static int clear(void *p, size_t bytes) {
    const int i = find(p);
    if (i < 0) return OK;
    if (blocks[i].bytes == stub_fail_zero_bytes && stub_fail_zero_times > 0) { --stub_fail_zero_times; return LAUNCH_FAILURE; }
    if (p == blocks[i].p && bytes >= blocks[i].bytes) blocks[i].zeroed = 1;
    return OK;
}

void **__hipRegisterFatBinary(const void *data) { static void *h; (void)data; return &h; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterFunction(void **m, const void *host, char *dev, const char *name, unsigned t, void *a, void *b, void *c, void *d, int *w) {
    (void)m; (void)dev; (void)t; (void)a; (void)b; (void)c; (void)d; (void)w;
    if (num_kernels < 4096) { kernels[num_kernels].host = host; snprintf(kernels[num_kernels].name, 256, "%s", name); ++num_kernels; }
}
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t s, int c, int g) { (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g; }
static dim3 cfg_g, cfg_b; static size_t cfg_s; static void *cfg_st;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, void *st) { cfg_g = g; cfg_b = b; cfg_s = s; cfg_st = st; return OK; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, void **st) { *g = cfg_g; *b = cfg_b; *s = cfg_s; *st = cfg_st; return OK; }
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t s, void *st) {
    (void)g; (void)b; (void)st;
    if (s > lds_allowed(f)) ++stub_lds_refused;
    const char *name = "";
    for (int i = 0; i < num_kernels; ++i) if (kernels[i].host == f) name = kernels[i].name;
    if (strstr(name, "k_fill_u32")) {
        const int rc = clear(*(void **)args[0], 4 * *(size_t *)args[1]);
        if (rc) last_error = rc;
        return rc;
    }
    if (stub_watch[0] && strstr(name, stub_watch)) {
        void *p = *(void **)args[stub_watch_arg];
        ++stub_watched;
        if (!p) ++stub_watched_null;
        else if (find(p) < 0 || !blocks[find(p)].zeroed) ++stub_watched_uncleared;
    }
    return OK;
}
int hipMalloc(void **p, size_t bytes) {
    stub_alloc_bytes[stub_allocs++ % 4096] = bytes;
    if (bytes == stub_fail_alloc_bytes) { ++stub_allocs_of_size; *p = NULL; last_error = OUT_OF_MEMORY; return OUT_OF_MEMORY; }
    *p = malloc(bytes ? bytes : 1);
    blocks[num_blocks].p = *p; blocks[num_blocks].bytes = bytes; blocks[num_blocks].zeroed = 0; ++num_blocks;
    return OK;
}
int hipFree(void *p) { ++stub_frees; const int i = find(p); if (i >= 0) blocks[i].p = NULL; free(p); return OK; }
int hipMemset(void *p, int v, size_t bytes) { (void)v; const int rc = clear(p, bytes); if (rc) last_error = rc; return rc; }
int hipMemsetAsync(void *p, int v, size_t bytes, void *st) { (void)st; return hipMemset(p, v, bytes); }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { (void)d; (void)s; (void)n; (void)k; (void)st; return OK; }
int hipGetLastError(void) { const int e = last_error; last_error = OK; return e; }
const char *hipGetErrorString(int e) { (void)e; return "stub"; }
int hipGetDevice(int *d) { *d = stub_device; return OK; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 65536; return OK; }
int hipGetSymbolAddress(void **p, const void *s) { (void)s; static char x[16]; *p = x; return OK; }
int hipDeviceSynchronize(void) { ++stub_device_syncs; return OK; }
int hipStreamSynchronize(void *st) { (void)st; ++stub_stream_syncs; return OK; }
int hipStreamCreateWithFlags(void **st, unsigned f) { (void)f; *st = malloc(1); return OK; }
int hipStreamDestroy(void *st) { free(st); return OK; }
int hipStreamWaitEvent(void *st, void *e, unsigned f) { (void)st; (void)e; (void)f; return OK; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; *e = malloc(1); return OK; }
int hipEventDestroy(void *e) { free(e); return OK; }
int hipEventRecord(void *e, void *st) { (void)e; (void)st; return OK; }
int hipFuncSetAttribute(const void *f, int a, int v) {
    (void)a;
    if (stub_lds_calls < 4096) { lds[stub_lds_calls].host = f; lds[stub_lds_calls].device = stub_device; lds[stub_lds_calls].bytes = (size_t)v; ++stub_lds_calls; }
    return OK;
}
