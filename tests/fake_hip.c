/* A stand-in for the HIP runtime with no GPU behind it: device memory is host
 * memory, kernels do not run, every launch is recorded.  A launch that forms a
 * state for a waiting host call (finalize_kernel, and the first flat_kernel of a
 * call) leaves words for the pinned block of the plan, stored at once or when
 * the "stream" is next found drained.  Knobs and counters are the fake_*
 * symbols; the driving side is fake_hip.py. */
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3;
typedef int hipError_t;
enum { OK = 0, NOT_READY = 600, LAUNCH_FAILURE = 719, UNKNOWN = 999, OUT_OF_MEMORY = 2 };

/* knobs */
int fake_fail_at = -1;        /* index of the launch that fails */
int fake_pending = 0;         /* 1: words and launches wait for a synchronisation */
int fake_queries = 0;         /* stream queries answered "not ready" before the work is done; -1: for ever */
int fake_query_limit = 1000;  /* more queries than this in one go: error */
int fake_s = 3;
double fake_dt_par = 1.0;
unsigned fake_flags = 0;      /* device flags (4: blocking synchronisation) */
int fake_cap_bytes_on = 0;    /* refuse allocations above fake_cap_bytes */
size_t fake_cap_bytes = 0;
/* counters */
int fake_unfinished = 0;      /* launches since the last synchronisation */
int fake_syncs = 0, fake_asked = 0;

#define MAXL 200000
static struct { const char *name; dim3 g, b; size_t lds; } rec[MAXL];
static int nrec, nlaunch;
static hipError_t last;
static struct { const void *f; const char *name; } fn[4096];
static int nfn;
static dim3 cg, cb;
static size_t cl;
static void *cs;
static unsigned char *words;  /* the plan's pinned block: double dt_par, int32 s */
static int have;

int fake_count(void) { return nrec; }
const char *fake_name(int i) { return rec[i].name; }
void fake_shape(int i, unsigned *o) { o[0] = rec[i].g.x; o[1] = rec[i].b.x; o[2] = (unsigned)rec[i].lds; }
void fake_reset(void) { nrec = nlaunch = 0; }

static void store(void) {
    if (have && words) {
        memcpy(words, &fake_dt_par, 8);
        memcpy(words + 8, &fake_s, 4);
    }
    have = 0;
}
static void drain(void) {
    store();
    fake_unfinished = 0;
    fake_asked = 0;
}
static const char *name_of(const void *f) {
    for (int i = 0; i < nfn; ++i)
        if (fn[i].f == f) return fn[i].name;
    return "?";
}

void **__hipRegisterFatBinary(const void *d) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **h) {}
void __hipRegisterFunction(void **h, const void *f, char *df, const char *name, unsigned l, void *a, void *b, void *c,
                           void *d, int *w) {
    fn[nfn].f = f;
    fn[nfn++].name = name;
}
void __hipRegisterVar(void **h, void *v, char *hv, char *dv, int e, size_t n, int c, int g) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, void *s) { cg = g; cb = b; cl = l; cs = s; return OK; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *l, void **s) { *g = cg; *b = cb; *l = cl; *s = cs; return OK; }

hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t lds, void *st) {
    const char *n = name_of(f);
    if (nlaunch++ == fake_fail_at) return last = LAUNCH_FAILURE;
    if (nrec < MAXL) { rec[nrec].name = n; rec[nrec].g = g; rec[nrec].b = b; rec[nrec++].lds = lds; }
    ++fake_unfinished;
    if (strstr(n, "finalize_kernel") || strstr(n, "flat_kernel")) {
        have = 1;
        if (!fake_pending) store();
    }
    return OK;
}

size_t fake_alloc[4096];      /* sizes of the device allocations, in order */
int fake_allocs = 0;
hipError_t hipMalloc(void **p, size_t n) {
    if (fake_allocs < 4096) fake_alloc[fake_allocs++] = n;
    if (fake_cap_bytes_on && n > fake_cap_bytes) { *p = NULL; return last = OUT_OF_MEMORY; }
    *p = aligned_alloc(256, (n + 255) / 256 * 256 + 256);   /* pages are touched only where written */
    return *p ? OK : (last = OUT_OF_MEMORY);
}
hipError_t hipFree(void *p) { free(p); return OK; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned f) { *p = calloc(1, n + 64); words = *p; return OK; }
hipError_t hipHostFree(void *p) { if (p == words) words = NULL; free(p); return OK; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, int k) { drain(); memcpy(d, s, n); return OK; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { return OK; }
hipError_t hipMemset(void *d, int v, size_t n) { memset(d, v, n); return OK; }
hipError_t hipDeviceSynchronize(void) { ++fake_syncs; drain(); return OK; }
hipError_t hipStreamSynchronize(void *s) { ++fake_syncs; drain(); return OK; }
hipError_t hipStreamQuery(void *s) {
    if (++fake_asked > fake_query_limit) return last = UNKNOWN;
    if (fake_pending && fake_unfinished && (fake_queries < 0 || fake_asked <= fake_queries)) return NOT_READY;
    drain();
    return OK;
}
hipError_t hipStreamIsCapturing(void *s, int *c) { *c = 0; return OK; }
hipError_t hipGetLastError(void) { hipError_t e = last; last = OK; return e; }
hipError_t hipPeekAtLastError(void) { return last; }
const char *hipGetErrorString(hipError_t e) { return "stand-in error"; }
hipError_t hipGetDevice(int *d) { *d = 0; return OK; }
hipError_t hipSetDevice(int d) { return OK; }
hipError_t hipGetDeviceFlags(unsigned *f) { *f = fake_flags; return OK; }
hipError_t hipDeviceGetAttribute(int *v, int a, int d) { *v = 256; return OK; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int b, size_t l) { *n = 3; return OK; }
hipError_t hipGetSymbolAddress(void **p, const void *s) {
    static void *mem;
    if (!mem) mem = aligned_alloc(256, 64u << 20);
    *p = mem;
    return OK;
}
/* events tick one launch at a time */
hipError_t hipEventCreate(void **e) { *e = calloc(1, 8); return OK; }
hipError_t hipEventDestroy(void *e) { free(e); return OK; }
hipError_t hipEventRecord(void *e, void *s) { *(int *)e = nlaunch; return OK; }
hipError_t hipEventSynchronize(void *e) { drain(); return OK; }
hipError_t hipEventElapsedTime(float *t, void *a, void *b) { *t = (float)(*(int *)b - *(int *)a); return OK; }
hipError_t hipStreamCreateWithFlags(void **s, unsigned f) { *s = (void *)16; return OK; }
hipError_t hipStreamDestroy(void *s) { return OK; }
hipError_t hipStreamBeginCapture(void *s, int m) { return OK; }
hipError_t hipStreamEndCapture(void *s, void **g) { *g = (void *)16; return OK; }
hipError_t hipGraphInstantiate(void **e, void *g, void *a, char *b, size_t n) { *e = (void *)16; return OK; }
hipError_t hipGraphLaunch(void *e, void *s) { return OK; }
hipError_t hipGraphExecDestroy(void *e) { return OK; }
hipError_t hipGraphDestroy(void *g) { return OK; }
