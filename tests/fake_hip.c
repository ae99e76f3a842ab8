/* A HIP runtime without a device, for tests of the library's host code: memory
 * is a number of bytes, kernels are not run, and every call that matters is
 * written to a log.  Loaded before the library, its functions take the place of
 * the runtime's. */
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

static char *text;
static size_t used, room;

static void say(const char *fmt, ...) {
    char line[512];
    va_list ap;
    va_start(ap, fmt);
    const size_t n = (size_t)vsnprintf(line, sizeof line, fmt, ap);
    va_end(ap);
    if (used + n + 2 > room) text = realloc(text, room = 2 * room + 4096);
    memcpy(text + used, line, n);
    used += n;
    text[used++] = '\n';
    text[used] = 0;
}

const char *fake_log(void) { return used ? text : ""; }
void fake_clear(void) { used = 0; }

static size_t free_bytes = (size_t)1 << 50;
static int fail_in = -1; /* the allocation after this many more fails */
void fake_memory(size_t bytes) { free_bytes = bytes; }
void fake_fail(int after) { fail_in = after; }

static struct { uintptr_t at; size_t size; } blocks[4096];
static int n_blocks;
static uintptr_t next_at = (uintptr_t)1 << 40;

hipError_t hipMalloc(void **p, size_t size) {
    const int fail = fail_in == 0 || size > free_bytes || n_blocks == 4096;
    if (fail_in >= 0) --fail_in;
    say("malloc %zu %s", size, fail ? "failed" : "ok");
    if (fail) return hipErrorOutOfMemory;
    free_bytes -= size;
    blocks[n_blocks].at = next_at;
    blocks[n_blocks++].size = size;
    *p = (void *)next_at;
    next_at += (size + 4095) & ~(size_t)4095;
    return hipSuccess;
}

hipError_t hipFree(void *p) {
    for (int i = 0; i < n_blocks; ++i)
        if (blocks[i].at == (uintptr_t)p) {
            say("free %zu", blocks[i].size);
            free_bytes += blocks[i].size;
            blocks[i] = blocks[--n_blocks];
            return hipSuccess;
        }
    return hipErrorInvalidValue;
}

size_t fake_blocks(void) { return (size_t)n_blocks; }

hipError_t hipHostMalloc(void **p, size_t size, unsigned int flags) {
    (void)flags;
    *p = calloc(1, size);
    return hipSuccess;
}

hipError_t hipMemset(void *p, int v, size_t n) {
    (void)p, (void)v;
    say("memset %zu stream 0", n);
    return hipSuccess;
}

hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind kind, hipStream_t st) {
    (void)s;
    say("copy %zu stream %p", n, (void *)st);
    if (kind == hipMemcpyDeviceToHost) memset(d, 0, n);
    return hipSuccess;
}

hipError_t hipStreamSynchronize(hipStream_t s) {
    say("sync %p", (void *)s);
    return hipSuccess;
}

hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipSetDevice(int d) { return d == 0 ? hipSuccess : hipErrorInvalidDevice; }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipGetDeviceCount(int *n) { return *n = 1, hipSuccess; }
static hipError_t last = hipSuccess;
hipError_t hipPeekAtLastError(void) { return last; }
hipError_t hipGetLastError(void) {
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}

const char *hipGetErrorString(hipError_t e) { return e == hipSuccess ? "success" : "error"; }
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute a, int v) { return (void)f, (void)a, (void)v, hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *s) { return *p = (void *)s, hipSuccess; }

hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int d) {
    (void)d;
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    return hipSuccess;
}

hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int block, size_t lds) {
    (void)f, (void)block, (void)lds;
    return *n = 4, hipSuccess;
}

/* kernels: the names from their registration, the launch from its call */
static struct { const void *host; const char *name; } kernels[4096];
static int n_kernels;

void **__hipRegisterFatBinary(const void *data) {
    static void *handle;
    (void)data;
    return &handle;
}

void __hipUnregisterFatBinary(void **modules) { (void)modules; }

void __hipRegisterFunction(void **modules, const void *host, char *dev, const char *name, unsigned int threads,
                           void *tid, void *bid, void *bdim, void *gdim, int *wsize) {
    (void)modules, (void)dev, (void)threads, (void)tid, (void)bid, (void)bdim, (void)gdim, (void)wsize;
    if (n_kernels < 4096) {
        kernels[n_kernels].host = host;
        kernels[n_kernels++].name = name;
    }
}

void __hipRegisterVar(void **modules, void *var, char *host, char *dev, int ext, size_t size, int constant, int global) {
    (void)modules, (void)var, (void)host, (void)dev, (void)ext, (void)size, (void)constant, (void)global;
}

static struct { dim3 grid, block; size_t lds; hipStream_t stream; } conf;

hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
    conf.grid = grid;
    conf.block = block;
    conf.lds = lds;
    conf.stream = stream;
    return hipSuccess;
}

hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *stream) {
    *grid = conf.grid;
    *block = conf.block;
    *lds = conf.lds;
    *stream = conf.stream;
    return hipSuccess;
}

hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t stream) {
    const char *name = "?";
    (void)args;
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i].host == f) name = kernels[i].name;
    say("launch %s grid %u %u block %u lds %zu stream %p", name, grid.x, grid.y, block.x, lds, (void *)stream);
    if ((uint64_t)grid.x * block.x <= 0xFFFFFFFFull) return hipSuccess;
    return last = hipErrorInvalidConfiguration; /* a grid's threads per axis fit 32 bits */
}
