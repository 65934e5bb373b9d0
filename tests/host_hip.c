/* host_hip.c -- a stand-in for the HIP runtime calls that libdr.so makes, for
 * tests of the library's host side without a GPU.  Preloaded into a process of
 * its own: "device" memory is host memory, kernels are counted and not run, and
 * the test sets what the runtime would report (a stream that is captured, a
 * card with little memory). */
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

enum { OK = 0, OUT_OF_MEMORY = 2, CAPTURE_UNSUPPORTED = 900 };
typedef struct { uint32_t x, y, z; } dim3_t;

/* ---- what the test sets and reads */
#define MAX_ALLOCS 4096
static struct { void* p; size_t bytes; } live[MAX_ALLOCS];
static int n_live;
static size_t used, room = (size_t)1 << 50;
static int capturing, violations, launches;
static uintptr_t streams[16];
static int n_streams;
static unsigned long long* pinned;

void fake_capture(int on) { capturing = on; }
void fake_room(size_t bytes) { room = bytes; }
size_t fake_used(void) { return used; }
int fake_violations(void) { return violations; }           /* calls that a capture does not allow */
unsigned long long* fake_pinned(void) { return pinned; }
int fake_live(void** out) {
    for (int i = 0; i < n_live; ++i) out[i] = live[i].p;
    return n_live;
}
void fake_reset_launches(void) { launches = n_streams = 0; }
int fake_launches(void) { return launches; }
int fake_streams(void) { return n_streams; }

static int not_captured(void) {
    if (!capturing) return OK;
    ++violations;
    return CAPTURE_UNSUPPORTED;
}

/* ---- memory */
int hipMalloc(void** p, size_t bytes) {
    int e = not_captured();
    if (e) return e;
    if (used + bytes > room || n_live == MAX_ALLOCS || !(*p = calloc(1, bytes ? bytes : 1))) return OUT_OF_MEMORY;
    live[n_live].p = *p;
    live[n_live++].bytes = bytes;
    used += bytes;
    return OK;
}

int hipFree(void* p) {
    int e = not_captured();
    if (e) return e;
    for (int i = 0; i < n_live; ++i)
        if (live[i].p == p) {
            used -= live[i].bytes;
            live[i] = live[--n_live];
            free(p);
            return OK;
        }
    return p ? 1 : OK;
}

int hipHostMalloc(void** p, size_t bytes, unsigned flags) {
    int e = not_captured();
    (void)flags;
    if (e) return e;
    *p = calloc(1, bytes);
    pinned = (unsigned long long*)*p;
    return OK;
}

int hipHostFree(void* p) { free(p); return OK; }
int hipMemcpy(void* d, const void* s, size_t n, int k) { (void)k; memcpy(d, s, n); return OK; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { (void)st; return hipMemcpy(d, s, n, k); }
/* (allocations start at zero and no kernel writes them) */
int hipMemset(void* d, int v, size_t n) { (void)d; (void)v; (void)n; return OK; }
int hipMemsetAsync(void* d, int v, size_t n, void* st) { (void)st; return hipMemset(d, v, n); }
int hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = (void*)0x100000; return OK; }

/* ---- device, streams, events */
int hipGetDevice(int* d) { *d = 0; return OK; }
int hipSetDevice(int d) { (void)d; return OK; }
int hipGetLastError(void) { return OK; }
int hipStreamSynchronize(void* st) { (void)st; return not_captured(); }
int hipStreamCreateWithFlags(void** st, unsigned f) { (void)f; *st = malloc(1); return OK; }
int hipStreamDestroy(void* st) { free(st); return OK; }
int hipStreamIsCapturing(void* st, int* s) { (void)st; *s = capturing ? 1 : 0; return OK; }
int hipStreamWaitEvent(void* st, void* ev, unsigned f) { (void)st; (void)ev; (void)f; return OK; }
int hipEventCreate(void** ev) { *ev = malloc(1); return OK; }
int hipEventCreateWithFlags(void** ev, unsigned f) { (void)f; return hipEventCreate(ev); }
int hipEventRecord(void* ev, void* st) { (void)ev; (void)st; return OK; }
int hipEventQuery(void* ev) { (void)ev; return OK; }
int hipEventDestroy(void* ev) { free(ev); return OK; }

/* ---- launches */
static dim3_t grid_, block_;
static size_t shared_;
static void* stream_;

int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t sh, void* st) {
    grid_ = g; block_ = b; shared_ = sh; stream_ = st;
    return OK;
}

int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* sh, void** st) {
    *g = grid_; *b = block_; *sh = shared_; *st = stream_;
    return OK;
}

int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** args, size_t sh, void* st) {
    (void)f; (void)g; (void)b; (void)args; (void)sh;
    ++launches;
    int i = 0;
    while (i < n_streams && streams[i] != (uintptr_t)st) ++i;
    if (i == n_streams && n_streams < 16) streams[n_streams++] = (uintptr_t)st;
    return OK;
}
