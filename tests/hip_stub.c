/* A HIP runtime that runs nothing, for host-side tests of libnt without a GPU: memory is host memory, copies are copies,
 * a kernel launch is written down (kernel, grid) and does no work.  Loaded with RTLD_GLOBAL before libnt.so, so that the
 * library's runtime calls bind to it.  stub_event_status is what every event reports. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <unistd.h>

typedef struct { uint32_t x, y, z; } dim3;
enum { OK = 0, NOT_READY = 600 };

int stub_event_status = OK;
int stub_slow_limits = 0;

/* launches */
enum { MAX_FUNCS = 4096, MAX_LAUNCHES = 1 << 16 };
static struct { const void *f; const char *name; int lds; } funcs[MAX_FUNCS];  /* lds: dynamic LDS a launch may ask for */
static int n_funcs = 0;
static struct { const char *name; dim3 grid; } launches[MAX_LAUNCHES];
static int n_launches = 0;

int stub_n_funcs(void) { return n_funcs; }
const char *stub_func(int i) { return funcs[i].name; }
void stub_clear(void) { n_launches = 0; }
int stub_n_launches(void) { return n_launches; }
const char *stub_launch(int i, uint32_t grid[3]) {
  grid[0] = launches[i].grid.x, grid[1] = launches[i].grid.y, grid[2] = launches[i].grid.z;
  return launches[i].name;
}

static void *module_handle;
void **__hipRegisterFatBinary(const void *data) { return &module_handle; }
void __hipUnregisterFatBinary(void **m) {}
void __hipRegisterFunction(void **m, const void *f, char *df, const char *name, unsigned limit, void *t, void *b, dim3 *bd,
                           dim3 *gd, int *ws) {
  if (strncmp(name, "_ZN2nt", 6)) return; /* other libraries' kernels */
  if (n_funcs < MAX_FUNCS) funcs[n_funcs].f = f, funcs[n_funcs].name = strdup(name), funcs[n_funcs].lds = 64 * 1024, n_funcs++;
}
void __hipRegisterVar(void **m, void *var, char *hv, char *dv, int ext, size_t size, int constant, int global) {}

static __thread struct { dim3 grid, block; size_t lds; void *stream; } config;
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *stream) {
  config.grid = grid, config.block = block, config.lds = lds, config.stream = stream;
  return OK;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream) {
  *grid = config.grid, *block = config.block, *lds = config.lds, *stream = config.stream;
  return OK;
}
static __thread int last_error;
int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, void *stream) {
  int at = __atomic_fetch_add(&n_launches, 1, __ATOMIC_SEQ_CST);
  if (at >= MAX_LAUNCHES) abort();
  launches[at].grid = grid, launches[at].name = "?";
  for (int i = 0; i < n_funcs; i++)
    if (funcs[i].f == f) {
      launches[at].name = funcs[i].name;
      if (lds > (size_t)__atomic_load_n(&funcs[i].lds, __ATOMIC_SEQ_CST)) return last_error = 1;
    }
  return OK;
}
/* the dynamic LDS limit (the one attribute in use).  With stub_slow_limits the smallest of several values set at a time takes
 * effect last and returns first. */
int hipFuncSetAttribute(const void *f, int attr, int value) {
  const int slow = stub_slow_limits && value < 160 * 1024;
  if (slow) usleep(160 * 1024 - value);
  for (int i = 0; i < n_funcs; i++)
    if (funcs[i].f == f) __atomic_store_n(&funcs[i].lds, value, __ATOMIC_SEQ_CST);
  if (slow && value > 80 * 1024) usleep(2 * value - 160 * 1024);
  return OK;
}

int hipMalloc(void **p, size_t n) { return (*p = calloc(n ? n : 1, 1)) ? OK : 2; }
int hipFree(void *p) { free(p); return OK; }
int hipHostMalloc(void **p, size_t n, unsigned flags) { return hipMalloc(p, n); }
int hipHostFree(void *p) { return hipFree(p); }
int hipHostGetDevicePointer(void **d, void *h, unsigned flags) { *d = h; return OK; }
int64_t stub_copied = 0;
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *stream) { memmove(d, s, n); stub_copied += n; return OK; }
int hipMemsetAsync(void *d, int v, size_t n, void *stream) { return OK; } /* used on fresh memory only, which is zero */
int hipGetSymbolAddress(void **p, const void *s) { *p = &module_handle; return OK; }

int hipStreamCreateWithFlags(void **s, unsigned flags) { return hipMalloc(s, 1); }
int hipStreamDestroy(void *s) { return hipFree(s); }
int hipStreamSynchronize(void *s) { return stub_event_status == NOT_READY ? OK : stub_event_status; }
int hipStreamWaitEvent(void *s, void *e, unsigned flags) { return OK; }
int hipEventCreate(void **e) { return hipMalloc(e, 1); }
int hipEventCreateWithFlags(void **e, unsigned flags) { return hipMalloc(e, 1); }
int hipEventDestroy(void *e) { return hipFree(e); }
int hipEventRecord(void *e, void *s) { return OK; }
int hipEventElapsedTime(float *ms, void *a, void *b) { *ms = 1.f; return OK; }
int hipEventQuery(void *e) { return stub_event_status; }
int hipEventSynchronize(void *e) { return stub_event_status == NOT_READY ? OK : stub_event_status; }

int hipGetDevice(int *d) { *d = 0; return OK; }
int hipSetDevice(int d) { return OK; }
int hipGetLastError(void) { int e = last_error; last_error = OK; return e; }
const char *hipGetErrorString(int e) { return e == OK ? "no error" : "stub error"; }
