/* A stand-in for the HIP runtime on the CPU, for tests of the library's host code: "device" memory
 * is host memory, asynchronous copies are carried out when their stream is next waited for, kernels
 * are noted and not run.  Loaded with RTLD_GLOBAL before the library, it takes the place of the
 * runtime's functions.  The host side of a copy that has changed, or is no longer mapped, by then
 * counts as stale. */
#define _GNU_SOURCE
#include <stdlib.h>
#include <string.h>
#include <sys/uio.h>
#include <unistd.h>

typedef struct { unsigned x, y, z; } dim3_;
typedef struct { void* dst; const void* src; void* was; size_t n; } Copy;
typedef struct { unsigned grid, block; void* arg0; } Launch;

static Copy pending[4096];
static Launch launches[65536];
int standin_pending, standin_stale, standin_waits, standin_launches, standin_fail_malloc, standin_fail_copy;

const Launch* standin_launch(int i) { return &launches[i]; }

static void settle(void) {
  for (int i = 0; i < standin_pending; ++i) {
    Copy* c = &pending[i];
    char* now = malloc(c->n);
    struct iovec l = {now, c->n}, r = {(void*)c->src, c->n};
    if (process_vm_readv(getpid(), &l, 1, &r, 1, 0) != (ssize_t)c->n || memcmp(now, c->was, c->n)) ++standin_stale;
    memcpy(c->dst, c->was, c->n);
    free(now);
    free(c->was);
  }
  standin_pending = 0;
}

int hipGetDevice(int* d) { return *d = 0; }
int hipGetLastError(void) { return 0; }
const char* hipGetErrorString(int e) { return e ? "error" : "ok"; }
int hipMalloc(void** p, size_t n) {
  if (standin_fail_malloc && --standin_fail_malloc == 0) return 2;
  return (*p = calloc(1, n)) ? 0 : 2;
}
int hipFree(void* p) { free(p); return 0; }
int hipHostMalloc(void** p, size_t n, unsigned f) { return (*p = calloc(1, n)) ? 0 : 2; }
int hipHostFree(void* p) { free(p); return 0; }
int hipHostGetDevicePointer(void** d, void* h, unsigned f) { *d = h; return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int kind) { settle(); memmove(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* st) {
  if (standin_fail_copy && --standin_fail_copy == 0) return 1;
  if (kind != 1 || standin_pending == 4096) { settle(); memmove(d, s, n); return 0; }
  Copy c = {d, s, malloc(n), n};
  memcpy(c.was, s, n);
  pending[standin_pending++] = c;
  return 0;
}
int hipGetSymbolAddress(void** p, const void* s) { static char scratch[64 << 20]; *p = scratch; return 0; }
int hipStreamSynchronize(void* st) { ++standin_waits; settle(); return 0; }
int hipStreamIsCapturing(void* st, int* s) { return *s = 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { *s = malloc(1); return 0; }
int hipStreamDestroy(void* s) { free(s); return 0; }
int hipEventCreate(void** e) { *e = malloc(1); return 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { *e = malloc(1); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void* e, void* s) { return 0; }
int hipEventSynchronize(void* e) { ++standin_waits; settle(); return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { *ms = 1.f; return 0; }
int hipFuncSetAttribute(const void* f, int a, int v) { return 0; }
static struct { dim3_ grid, block; size_t lds; void* st; } conf;
int __hipPushCallConfiguration(dim3_ grid, dim3_ block, size_t lds, void* st) {
  conf.grid = grid; conf.block = block; conf.lds = lds; conf.st = st;
  return 0;
}
int __hipPopCallConfiguration(dim3_* grid, dim3_* block, size_t* lds, void** st) {
  *grid = conf.grid; *block = conf.block; *lds = conf.lds; *st = conf.st;
  return 0;
}
int hipLaunchKernel(const void* f, dim3_ grid, dim3_ block, void** args, size_t lds, void* st) {
  if (standin_launches < 65536) launches[standin_launches] = (Launch){grid.x, block.x, *(void**)args[0]};
  ++standin_launches;
  return 0;
}
