/* A HIP runtime on the host, for tests of what the library asks of one: it
 * allocates host memory, runs no kernel and keeps a log of the calls.  Loaded into
 * the global scope before liblbm_hip.so, whose references then bind to it.
 *
 * log lines: "launch KERNEL GRID BLOCK LDS" (mangled name), "malloc BYTES", "free",
 * "hostmalloc BYTES", "hostfree", "copy", "sync".
 * host_fail_launch(n): the n-th launch from now on (0 = the next) reports an error,
 * and is not logged. */
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef int hipError_t;
typedef struct { unsigned x, y, z; } dim3_t;

static char* g_log;
static size_t g_len, g_cap;
static void put(const char* fmt, ...) {
    char line[512];
    va_list ap;
    va_start(ap, fmt);
    const int n = vsnprintf(line, sizeof line, fmt, ap);
    va_end(ap);
    if (g_len + (size_t)n + 2 > g_cap) {
        g_cap = 2 * (g_len + (size_t)n + 2);
        g_log = realloc(g_log, g_cap);
    }
    memcpy(g_log + g_len, line, (size_t)n);
    g_len += (size_t)n;
    g_log[g_len++] = '\n';
    g_log[g_len] = 0;
}
const char* host_log(void) { return g_log ? g_log : ""; }
void host_log_clear(void) {
    g_len = 0;
    if (g_log) g_log[0] = 0;
}

static long g_fail = -1;
static hipError_t g_last;
void host_fail_launch(long n) { g_fail = n; }

/* kernels by the address of their host stub */
#define MAX_KERNELS 4096
static struct { const void* stub; char name[240]; } g_kernels[MAX_KERNELS];
static unsigned slot_of(const void* stub) {
    unsigned i = (unsigned)((size_t)stub >> 4) % MAX_KERNELS;
    while (g_kernels[i].stub && g_kernels[i].stub != stub) i = (i + 1) % MAX_KERNELS;
    return i;
}
void** __hipRegisterFatBinary(const void* data) {
    static void* handle;
    (void)data;
    return &handle;
}
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* stub, char* dev, const char* name, unsigned limit,
                           void* tid, void* bid, void* bdim, void* gdim, int* wsize) {
    (void)m, (void)dev, (void)limit, (void)tid, (void)bid, (void)bdim, (void)gdim, (void)wsize;
    const unsigned i = slot_of(stub);
    g_kernels[i].stub = stub;
    snprintf(g_kernels[i].name, sizeof g_kernels[i].name, "%s", name);
}
void __hipRegisterVar(void** m, void* var, char* host, char* name, int ext, size_t size, int c,
                      int global) {
    (void)m, (void)var, (void)host, (void)name, (void)ext, (void)size, (void)c, (void)global;
}

static struct { dim3_t grid, block; size_t lds; void* stream; } g_call;
hipError_t __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void* stream) {
    g_call.grid = grid, g_call.block = block, g_call.lds = lds, g_call.stream = stream;
    return 0;
}
hipError_t __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* lds, void** stream) {
    *grid = g_call.grid, *block = g_call.block, *lds = g_call.lds, *stream = g_call.stream;
    return 0;
}
hipError_t hipLaunchKernel(const void* stub, dim3_t grid, dim3_t block, void** args, size_t lds,
                           void* stream) {
    (void)args, (void)stream;
    if (g_fail >= 0 && g_fail-- == 0) return g_last = 719;
    put("launch %s %u %u %zu", g_kernels[slot_of(stub)].name, grid.x * grid.y * grid.z, block.x * block.y * block.z, lds);
    return 0;
}
hipError_t hipGetLastError(void) {
    const hipError_t e = g_last;
    g_last = 0;
    return e;
}
const char* hipGetErrorString(hipError_t e) { return e ? "launch failure" : "no error"; }

hipError_t hipMalloc(void** p, size_t n) {
    put("malloc %zu", n);
    *p = malloc(n ? n : 1);
    return *p ? 0 : 2;
}
hipError_t hipFree(void* p) {
    put("free");
    free(p);
    return 0;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned flags) {
    (void)flags;
    put("hostmalloc %zu", n);
    *p = calloc(1, n ? n : 1);
    return *p ? 0 : 2;
}
hipError_t hipHostFree(void* p) {
    put("hostfree");
    free(p);
    return 0;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, int kind) {
    (void)d, (void)s, (void)n, (void)kind;
    return 0;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* st) {
    (void)d, (void)s, (void)n, (void)kind, (void)st;
    put("copy");
    return 0;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, void* st) {
    (void)d, (void)v, (void)n, (void)st;
    return 0;
}
hipError_t hipStreamSynchronize(void* st) {
    (void)st;
    put("sync");
    return 0;
}
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return 0;
}
hipError_t hipDeviceGetAttribute(int* v, int attr, int dev) {
    (void)attr, (void)dev;
    *v = 256; /* only the number of compute units is asked for */
    return 0;
}
hipError_t hipGetSymbolAddress(void** p, const void* sym) {
    static double table[8];
    (void)sym;
    *p = table;
    return 0;
}
hipError_t hipStreamCreateWithFlags(void** st, unsigned flags) {
    static int stream;
    (void)flags;
    *st = &stream;
    return 0;
}
hipError_t hipStreamDestroy(void* st) {
    (void)st;
    return 0;
}
