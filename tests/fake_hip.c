/* A HIP runtime of host memory that launches nothing, for tests of the library's host code on machines without a GPU:
 * which kernels a call launches on which stream and buffers, what it allocates, and what it answers when a runtime call
 * fails.  Loaded under the runtime's own library name in a process of its own (test_host_routes.py).  hipGetLastError
 * returns the last error of any call of this thread and clears it; calls that succeed leave it alone. */
#define _GNU_SOURCE
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

#define BIG ((size_t)1 << 30)
enum { OK = 0, INVALID = 1, NOMEM = 2, IMPLICIT = 906 /* hipErrorStreamCaptureImplicit */, NOTREADY = 600 };
enum { K_LAUNCH = 0, K_MALLOC = 1, K_WAIT = 2, K_RECORD = 3 };
typedef struct {
    int kind;
    unsigned grid[3];
    void* stream;
    const void *in, *out;  /* launches of one layer: its input and output */
    int flags;             /* ... and how these lie: the kernel's own flags (test_host_routes.py) */
    char name[160];
} Entry;
typedef struct {
    int done, used;
} Event;
typedef struct {
    unsigned x, y, z;
} Dim3;

static _Thread_local int last_error;
static int fail_mallocs, fail_capture_query, fail_attributes, live;
static Entry logged[4096];
static int entries;
static uintptr_t capturing_stream = ~(uintptr_t)0, busy[64];
static int n_busy;
static Event* events[256];
static int n_events;
static struct {
    const void* host;
    char name[160];
} kernels[1024];
static int n_kernels;
static struct {
    void* at;
    size_t size;
} maps[256];
static int n_maps;

static int ret(int e) {
    if (e) last_error = e;
    return e;
}
static Entry* add(int kind, void* stream) {
    static Entry spill;
    Entry* e = entries < 4096 ? &logged[entries++] : &spill;
    memset(e, 0, sizeof(*e));
    e->kind = kind;
    e->stream = stream;
    return e;
}
static int is_busy(void* s) {
    for (int i = 0; i < n_busy; ++i)
        if (busy[i] == (uintptr_t)s) return 1;
    return 0;
}

/* ---- what the test sets and reads */
void fake_fail_mallocs(int on) { fail_mallocs = on; }
void fake_fail_capture_query(int on) { fail_capture_query = on; }
void fake_fail_attributes(int on) { fail_attributes = on; }
void fake_capture(uintptr_t s) { capturing_stream = s; }
void fake_set_busy(uintptr_t s) { busy[n_busy++ & 63] = s; }
void fake_finish_all(void) {
    n_busy = 0;
    for (int i = 0; i < n_events; ++i) events[i]->done = 1;
}
void fake_clear(void) { entries = 0; }
int fake_entries(void) { return entries; }
const Entry* fake_entry(int i) { return &logged[i]; }
int fake_live(void) { return live; }

/* ---- the runtime */
int hipGetLastError(void) {
    int e = last_error;
    last_error = 0;
    return e;
}
int hipMalloc(void** p, size_t n) {
    add(K_MALLOC, NULL);
    if (fail_mallocs) return ret(NOMEM);
    if (n > BIG) { /* addresses without memory behind them: nothing runs that would touch it */
        *p = mmap(NULL, n, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
        if (*p == MAP_FAILED) return ret(NOMEM);
        if (n_maps < 256) maps[n_maps].at = *p, maps[n_maps++].size = n;
    } else {
        *p = aligned_alloc(256, (n + 255) / 256 * 256);
    }
    ++live;
    return ret(*p ? OK : NOMEM);
}
int hipHostMalloc(void** p, size_t n, unsigned f) {
    (void)f;
    return hipMalloc(p, n);
}
int hipFree(void* p) {
    if (p) --live;
    for (int i = 0; i < n_maps; ++i)
        if (maps[i].at == p) {
            munmap(p, maps[i].size);
            maps[i] = maps[--n_maps];
            return OK;
        }
    free(p);
    return OK;
}
int hipHostFree(void* p) { return hipFree(p); }
int hipHostGetDevicePointer(void** d, void* h, unsigned f) {
    (void)f;
    *d = h;
    return OK;
}
int hipMemset(void* p, int v, size_t n) {
    memset(p, v, n);
    return OK;
}
int hipMemcpy(void* d, const void* s, size_t n, int k) {
    (void)k;
    memcpy(d, s, n);
    return OK;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) {
    (void)st;
    return hipMemcpy(d, s, n, k);
}
int hipDeviceSynchronize(void) { return OK; }
int hipStreamSynchronize(void* s) { (void)s; return OK; }
int hipStreamQuery(void* s) { (void)s; return OK; }
int hipGetDevice(int* d) { *d = 0; return OK; }
int hipGetDeviceCount(int* n) { *n = 1; return OK; }
int hipFuncSetAttribute(const void* f, int a, int v) {
    (void)f; (void)a; (void)v;
    return ret(fail_attributes ? INVALID : OK);
}
int hipGetSymbolAddress(void** p, const void* sym) {
    static char mem[17 << 20] __attribute__((aligned(256)));
    (void)sym;
    *p = mem;
    return OK;
}
int hipThreadExchangeStreamCaptureMode(int* m) { (void)m; return OK; }
int hipStreamIsCapturing(void* s, int* st) {
    if (fail_capture_query) return ret(IMPLICIT);
    *st = (uintptr_t)s == capturing_stream;
    return OK;
}
int hipEventCreateWithFlags(void** e, unsigned f) {
    (void)f;
    if (fail_mallocs) return ret(NOMEM);
    Event* v = calloc(1, sizeof(Event));
    v->done = 1;
    if (n_events < 256) events[n_events++] = v;
    *e = v;
    ++live;
    return OK;
}
int hipEventDestroy(void* e) { (void)e; --live; return OK; } /* (kept: fake_finish_all walks them) */
int hipEventRecord(void* e, void* s) {
    Event* v = e;
    v->used = 1;
    v->done = !is_busy(s);
    add(K_RECORD, s)->in = e;
    return OK;
}
int hipEventQuery(void* e) { return ((Event*)e)->done ? OK : ret(NOTREADY); }
int hipStreamWaitEvent(void* s, void* e, unsigned f) {
    (void)f;
    add(K_WAIT, s)->in = e;
    return OK;
}

static Dim3 push_grid, push_block;
static size_t push_shared;
static void* push_stream;
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t shared, void* s) {
    push_grid = g;
    push_block = b;
    push_shared = shared;
    push_stream = s;
    return OK;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* shared, void** s) {
    *g = push_grid;
    *b = push_block;
    *shared = push_shared;
    *s = push_stream;
    return OK;
}
int hipLaunchKernel(const void* f, Dim3 g, Dim3 b, void** args, size_t shared, void* s) {
    (void)shared;
    if ((unsigned long long)g.x * b.x > 0xffffffffull) return ret(INVALID); /* as the runtime: 2^32 threads along x */
    Entry* e = add(K_LAUNCH, s);
    e->grid[0] = g.x;
    e->grid[1] = g.y;
    e->grid[2] = g.z;
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i].host == f) strcpy(e->name, kernels[i].name);
    if (strstr(e->name, "k_layer_skinny") || strstr(e->name, "k_layer_rows")) { /* one struct: words 5 and 6, the last int */
        e->in = ((const void* const*)args[0])[5];
        e->out = ((const void* const*)args[0])[6];
        e->flags = ((const int*)args[0])[strstr(e->name, "k_layer_rows") ? 21 : 19];
    } else if (strstr(e->name, "k_layer_int8")) { /* LayerIO: in, out, LayerNorm rows, last layer's rows, two flags */
        e->in = ((const void* const*)args[3])[0];
        e->out = ((const void* const*)args[3])[1];
        e->flags = ((const int*)args[3])[8] | ((const int*)args[3])[9];
    } else if (strstr(e->name, "k_ln_tanh_rows") || strstr(e->name, "k_ln_tanh_long")) {
        e->in = *(const void* const*)args[0];
        e->out = *(const void* const*)args[8];
        e->flags = *(const long long*)args[9] != 0; /* 16-row tiles of a map in operand order */
    }
    return OK;
}
void** __hipRegisterFatBinary(const void* d) {
    static void* h;
    (void)d;
    return &h;
}
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned l, void* t, void* bid, void* bd, void* gd, int* w) {
    (void)m; (void)dev; (void)l; (void)t; (void)bid; (void)bd; (void)gd; (void)w;
    if (n_kernels == 1024) return;
    kernels[n_kernels].host = host;
    strncpy(kernels[n_kernels++].name, name, 159);
}
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t n, int c, int g) {
    (void)m; (void)v; (void)h; (void)d; (void)e; (void)n; (void)c; (void)g;
}
void __hipUnregisterFatBinary(void** m) { (void)m; }
