/* A stand-in for the HIP runtime on a machine without a GPU, for tests of the library's host logic: device memory is host memory,
 * kernels are not run, every call is written to a log, and a test can make the n-th call of a kind fail.  Loaded with its symbols
 * global before the library, so that the library's calls come here. */
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
enum { FAIL_CODE = 2 /* hipErrorOutOfMemory */, LOG_BYTES = 1 << 22 };

static char log_text[LOG_BYTES];
static size_t log_at;
static char fail_name[64];
static long fail_nth;
static int capturing, rows_all, rows_x1, last_error;
static struct { const void* host; char name[64]; } kernels[256];
static int n_kernels;
static struct { dim3 grid, block; size_t shared; void* stream; } config;

void hip_stub_clear(void) { log_at = 0; log_text[0] = 0; }
const char* hip_stub_log(void) { return log_text; }
void hip_stub_fail(const char* name, long nth) { snprintf(fail_name, sizeof fail_name, "%s", name); fail_nth = nth; }
void hip_stub_capturing(int on) { capturing = on; }
void hip_stub_rows(int all, int x1) { rows_all = all; rows_x1 = x1; } /* what a hand-off says of every expert */

static int call(const char* name, const char* fmt, ...) {
  const int failed = fail_nth > 0 && !strcmp(name, fail_name) && --fail_nth == 0;
  if (log_at + 512 < LOG_BYTES) {
    log_at += snprintf(log_text + log_at, 128, "%s ", name);
    va_list ap;
    va_start(ap, fmt);
    log_at += vsnprintf(log_text + log_at, 256, fmt, ap);
    va_end(ap);
    log_at += snprintf(log_text + log_at, 64, "%s\n", failed ? " FAILED" : "");
  }
  if (failed) last_error = FAIL_CODE;
  return failed ? FAIL_CODE : 0;
}

void** __hipRegisterFatBinary(const void* data) { static void* handle; (void)data; return &handle; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t s, int c, int g) { (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g; }
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned l, void* t, void* b, void* bd, void* gd, int* w) {
  (void)m; (void)dev; (void)l; (void)t; (void)b; (void)bd; (void)gd; (void)w;
  if (n_kernels == 256) abort();
  /* the kernels are in an anonymous namespace: ..._GLOBAL__N_1<length><name>... */
  const char* at = strstr(name, "_GLOBAL__N_1");
  char* k = NULL;
  const long n = at ? strtol(at + 12, &k, 10) : 0;
  kernels[n_kernels].host = host;
  snprintf(kernels[n_kernels++].name, 64, "%.*s", (int)n, k ? k : "");
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, void* stream) {
  config.grid = grid; config.block = block; config.shared = shared; config.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, void** stream) {
  *grid = config.grid; *block = config.block; *shared = config.shared; *stream = config.stream;
  return 0;
}
int hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t shared, void* stream) {
  const char* name = "?";
  for (int i = 0; i < n_kernels; ++i)
    if (kernels[i].host == f) name = kernels[i].name;
  (void)block; (void)shared;
  if (!strcmp(name, "k_copy_piece")) return call(name, "%p -> %p, %d x 16 on %p", *(void**)args[0], *(void**)args[1], *(int*)args[2], stream);
  if (!strcmp(name, "k_fill_zero")) return call(name, "%p, %zu on %p", *(void**)args[0], *(size_t*)args[1], stream);
  if (!strcmp(name, "k_handoff")) {
    const int EX = *(int*)args[5];
    int32_t* counts = *(int32_t**)args[8];
    for (int e = 0; e < EX; ++e) { counts[e] = rows_all; counts[EX + e] = rows_x1; }
  }
  return call(name, "%u %u on %p", grid.x, grid.y, stream);
}

static int take(const char* name, void** p, size_t n) {
  *p = NULL;
  if (call(name, "%zu", n)) return FAIL_CODE;
  *p = calloc(n ? n : 1, 1);
  return *p ? 0 : FAIL_CODE;
}
int hipMalloc(void** p, size_t n) { return take("hipMalloc", p, n); }
int hipMallocAsync(void** p, size_t n, void* s) { (void)s; return take("hipMallocAsync", p, n); }
int hipHostMalloc(void** p, size_t n, unsigned f) { (void)f; return take("hipHostMalloc", p, n); }
int hipFree(void* p) { free(p); return 0; }
int hipFreeAsync(void* p, void* s) { (void)s; free(p); return 0; }
int hipHostFree(void* p) { free(p); return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int k) {
  (void)k;
  if (call("hipMemcpy", "%p -> %p, %zu", s, d, n) || !d || !s) return FAIL_CODE;
  memcpy(d, s, n);
  return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* stream) {
  (void)k;
  if (call("hipMemcpyAsync", "%p -> %p, %zu on %p", s, d, n, stream) || !d || !s) return FAIL_CODE;
  memcpy(d, s, n);
  return 0;
}
int hipMemset(void* d, int v, size_t n) { if (call("hipMemset", "%zu", n)) return FAIL_CODE; memset(d, v, n); return 0; }

static int handle(const char* name, void** h) { *h = NULL; if (call(name, "")) return FAIL_CODE; *h = malloc(1); return 0; }
int hipEventCreate(void** e) { return handle("hipEventCreate", e); }
int hipEventCreateWithFlags(void** e, unsigned f) { (void)f; return handle("hipEventCreateWithFlags", e); }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 0.f; return 0; }
int hipEventRecord(void* e, void* s) { return call("hipEventRecord", "%p on %p", e, s); }
int hipEventSynchronize(void* e) { return call("hipEventSynchronize", "%p", e); }
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; return handle("hipStreamCreateWithFlags", s); }
int hipStreamDestroy(void* s) { free(s); return 0; }
int hipStreamSynchronize(void* s) { return call("hipStreamSynchronize", "%p", s); }
int hipStreamWaitEvent(void* s, void* e, unsigned f) { (void)f; return call("hipStreamWaitEvent", "%p for %p", s, e); }
int hipStreamIsCapturing(void* s, int* status) { (void)s; *status = capturing; return 0; }
int hipDeviceSynchronize(void) { return call("hipDeviceSynchronize", ""); }
int hipSetDevice(int d) { (void)d; return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetDeviceCount(int* n) { *n = 1; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipFuncSetAttribute(const void* f, int a, int v) { (void)f; (void)a; (void)v; return 0; }
int hipFuncGetAttributes(void* a, const void* f) { (void)a; (void)f; return 0; } /* (the library passes zeros) */
int hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = NULL; return FAIL_CODE; }
int hipGetLastError(void) { const int e = last_error; last_error = 0; return e; }
const char* hipGetErrorString(int e) { return e ? "made to fail" : "no error"; }
