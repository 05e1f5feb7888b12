/* A stand-in for the HIP runtime on the host: device memory is host memory,
 * and a launch runs no kernel but leaves what the host code reads of its
 * results. Loaded before libmcpath.so, whose calls then resolve here, it lets
 * the CPU tests observe the library's queueing: which results it reads before
 * it has waited for them, and what it leaves in the queue when a call fails. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct {
    uint32_t x, y, z;
} dim3;

static struct {
    const void *fn;
    char name[256];
} kernels[2048];
static int n_kernels;

/* Stores that a queued kernel makes later than its first ones: they appear
 * when the host waits. */
static struct {
    uint64_t *to, value;
} late[64];
static int n_late;

/* The order statistic: results of the next finishing passes (SelectResult:
 * key, n_tail, tail_sum, end, done), the first with done = 0 where
 * stub_select_misses is 1. */
int stub_select_misses;
uint64_t stub_key;
double stub_n_tail, stub_tail_sum;

/* Launches and copies queued since the last wait. */
int stub_pending;
/* The stub_fail_at-th call (from 1) that can fail does; 0: none. Counts down. */
int stub_fail_at;
static int last_error;
static int fails(void) { return stub_fail_at > 0 && --stub_fail_at == 0; }

static void later(void *to, const void *value) {
    late[n_late].to = (uint64_t *)to;
    memcpy(&late[n_late++].value, value, 8);
}

static void ran(const char *name, dim3 grid, void **args) {
    const char *p = strstr(name, "final_merge_kernelILi");
    if (p) {                               /* partials, n_blocks, stride, out, clock */
        const int C = atoi(p + 21), M = 2 + C + C * (C + 1) / 2;
        double *out = *(double **)args[3];
        for (uint32_t b = 0; b < grid.x; ++b)
            for (int i = 0; i < M; ++i) out[b * M + i] = i == 0 ? 1000.0 : i == 1 ? 0.0 : 1.0;
    } else if (strstr(name, "select_finish_kernel")) {   /* x, n, state, list, partials, out */
        uint64_t *out = *(uint64_t **)args[5];
        const uint32_t done = stub_select_misses-- > 0 ? 0u : 1u;
        const uint64_t end = 0;
        memcpy(out + 4, &done, 4);
        if (done) {
            later(out, &stub_key);
            later(out + 1, &stub_n_tail);
            later(out + 2, &stub_tail_sum);
            later(out + 3, &end);
        }
    }
}

void **__hipRegisterFatBinary(const void *data) {
    static void *handle;
    (void)data;
    return &handle;
}
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterFunction(void **h, const void *fn, char *a, const char *name, unsigned l, void *t,
                           void *b, void *bd, void *gd, int *w) {
    (void)h, (void)a, (void)l, (void)t, (void)b, (void)bd, (void)gd, (void)w;
    if (n_kernels >= 2048) abort();
    kernels[n_kernels].fn = fn;
    strncpy(kernels[n_kernels++].name, name, 255);
}
void __hipRegisterVar(void **h, void *v, char *n, char *m, int e, size_t s, int c, int g) {
    (void)h, (void)v, (void)n, (void)m, (void)e, (void)s, (void)c, (void)g;
}

static struct {
    dim3 grid, block;
    size_t lds;
    void *stream;
} config;
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *stream) {
    config.grid = grid;
    config.block = block;
    config.lds = lds;
    config.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream) {
    *grid = config.grid;
    *block = config.block;
    *lds = config.lds;
    *stream = config.stream;
    return 0;
}
int hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t lds, void *stream) {
    (void)block, (void)lds, (void)stream;
    if (fails()) return last_error = 719;  /* hipErrorLaunchFailure */
    ++stub_pending;
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i].fn == fn) {
            ran(kernels[i].name, grid, args);
            return 0;
        }
    return 98;                             /* hipErrorInvalidDeviceFunction */
}
int hipStreamSynchronize(void *stream) {
    (void)stream;
    for (int i = 0; i < n_late; ++i) *late[i].to = late[i].value;
    n_late = stub_pending = 0;
    return 0;
}

int hipGetLastError(void) {
    const int e = last_error;
    last_error = 0;
    return e;
}
const char *hipGetErrorString(int e) { return e ? "error" : "no error"; }
int hipGetDeviceCount(int *n) {
    *n = 1;
    return 0;
}
int hipSetDevice(int d) { return d == 0 ? 0 : 101; }
int stub_clock_khz = 100000;               /* 0: not reported */
int hipDeviceGetAttribute(int *value, int attribute, int d) {
    (void)attribute, (void)d;
    *value = stub_clock_khz;
    return stub_clock_khz ? 0 : (last_error = 1);   /* hipErrorInvalidValue */
}
int hipGetSymbolAddress(void **p, const void *symbol) {
    static char scratch[4 << 20];
    (void)symbol;
    *p = scratch;
    return 0;
}
uint64_t stub_malloc_bytes;                /* device memory allocated so far */
int hipMalloc(void **p, size_t n) {
    if (fails()) return 2;                 /* hipErrorOutOfMemory */
    stub_malloc_bytes += n;
    return (*p = calloc(n, 1)) ? 0 : 2;
}
int hipFree(void *p) {
    free(p);
    return 0;
}
int hipHostMalloc(void **p, size_t n, unsigned flags) {
    (void)flags;
    if (fails()) return 2;
    return (*p = calloc(n, 1)) ? 0 : 2;
}
int hipHostFree(void *p) { return hipFree(p); }
int hipMemcpyAsync(void *to, const void *from, size_t n, int kind, void *stream) {
    (void)kind, (void)stream;
    if (fails()) return 719;
    ++stub_pending;
    memcpy(to, from, n);
    return 0;
}
int hipMemsetAsync(void *p, int v, size_t n, void *stream) {
    (void)stream;
    memset(p, v, n);
    return 0;
}
int hipStreamCreate(void **s) {
    static int dummy;
    *s = &dummy;
    return 0;
}
int hipStreamDestroy(void *s) {
    (void)s;
    return 0;
}
int hipEventCreate(void **e) { return hipStreamCreate(e); }
int hipEventDestroy(void *e) { return hipStreamDestroy(e); }
int hipEventRecord(void *e, void *s) {
    (void)e, (void)s;
    return fails() ? 719 : 0;
}
int hipEventElapsedTime(float *ms, void *a, void *b) {
    (void)a, (void)b;
    *ms = 0.f;
    return 0;
}
int hipFuncSetAttribute(const void *f, int a, int v) {
    (void)f, (void)a, (void)v;
    return fails() ? 719 : 0;
}
