/* A HIP runtime that runs nothing: it records every kernel launch and can make
 * one of them fail.  Preloaded into a process without a GPU, it lets the host
 * side of libfsest.so run whole calls.  An error stays until hipGetLastError
 * reads it, which clears it. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;

enum { kMaxKernels = 4096, kMaxLaunches = 1 << 16, kLaunchFailure = 719, kBadConfiguration = 9 };

static struct { const void* host; const char* name; } kernels[kMaxKernels];
static int n_kernels;
static struct { int kernel; dim3_t grid, block; } launches[kMaxLaunches];
static int n_launches, fail_at = -1, last_error, occupancy_queries, elapsed_calls;
static struct { dim3_t grid, block; size_t lds; void* stream; } pushed;

/* ---- read and set by the test */
int stub_kernels(void) { return n_kernels; }
const char* stub_kernel(int i) { return kernels[i].name; }
int stub_launches(void) { return n_launches; }
const char* stub_launched(int i) { return kernels[launches[i].kernel].name; }
uint32_t stub_grid(int i, int axis) { return ((uint32_t*)&launches[i].grid)[axis]; }
uint32_t stub_block(int i) { return launches[i].block.x; }
int stub_occupancy_queries(void) { return occupancy_queries; }
/* forgets the launches; launch number at (from 0) of the following ones fails */
void stub_reset(int at) { n_launches = 0; fail_at = at; last_error = 0; occupancy_queries = 0; }

/* ---- code objects */
static void* module;
void** __hipRegisterFatBinary(const void* data) { (void)data; return &module; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterVar(void** m, void* v, char* a, char* b, int c, size_t d, int e, int f) {
  (void)m, (void)v, (void)a, (void)b, (void)c, (void)d, (void)e, (void)f;
}
void __hipRegisterFunction(void** m, const void* host, char* a, const char* name, unsigned l, void* t, void* b,
                           void* bd, void* gd, int* w) {
  (void)m, (void)a, (void)l, (void)t, (void)b, (void)bd, (void)gd, (void)w;
  if (!strstr(name, "5fsest")) return; /* other libraries' kernels */
  if (n_kernels < kMaxKernels) kernels[n_kernels].host = host, kernels[n_kernels++].name = name;
}

/* ---- launches */
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void* stream) {
  pushed.grid = grid, pushed.block = block, pushed.lds = lds, pushed.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* lds, void** stream) {
  *grid = pushed.grid, *block = pushed.block, *lds = pushed.lds, *stream = pushed.stream;
  return 0;
}
int hipLaunchKernel(const void* host, dim3_t grid, dim3_t block, void** args, size_t lds, void* stream) {
  (void)args, (void)stream;
  int k = 0;
  while (k < n_kernels && kernels[k].host != host) ++k;
  if (k == n_kernels || n_launches == kMaxLaunches) return last_error = kLaunchFailure;
  const int at = n_launches++;
  launches[at].kernel = k, launches[at].grid = grid, launches[at].block = block;
  if (at == fail_at) return last_error = kLaunchFailure;
  const uint64_t threads = (uint64_t)block.x * block.y * block.z;
  if (!grid.x || !grid.y || !grid.z || grid.y > 65535 || grid.z > 65535 || !threads || threads > 1024 ||
      lds > 160 * 1024)
    return last_error = kBadConfiguration;
  return 0;
}
int hipGetLastError(void) { const int e = last_error; last_error = 0; return e; }
const char* hipGetErrorString(int e) { return e ? "stub error" : "no error"; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int threads, size_t lds) {
  (void)f, (void)threads, (void)lds;
  ++occupancy_queries;
  *n = 2;
  return 0;
}
int hipFuncSetAttribute(const void* f, int a, int v) { (void)f, (void)a, (void)v; return 0; }

/* ---- device, memory (host memory stands for the device's), streams, graphs, events */
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipSetDevice(int d) { (void)d; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { (void)a, (void)d; *v = 256; return 0; }
int hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = (void*)(uintptr_t)(1 << 20); return 0; }
int hipMemcpyAsync(void* dst, const void* src, size_t n, int kind, void* s) {
  (void)kind, (void)s;
  memcpy(dst, src, n);
  return 0;
}
int hipStreamSynchronize(void* s) { (void)s; return 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = &module; return 0; }
int hipStreamDestroy(void* s) { (void)s; return 0; }
int hipStreamBeginCapture(void* s, int m) { (void)s, (void)m; return 0; }
int hipStreamEndCapture(void* s, void** g) { (void)s; *g = &module; return 0; }
int hipGraphInstantiate(void** e, void* g, void* n, char* b, size_t z) {
  (void)g, (void)n, (void)b, (void)z;
  *e = &module;
  return 0;
}
int hipGraphLaunch(void* e, void* s) { (void)e, (void)s; return 0; }
int hipGraphDestroy(void* g) { (void)g; return 0; }
int hipGraphExecDestroy(void* e) { (void)e; return 0; }
int hipEventCreate(void** e) { *e = &module; return 0; }
int hipEventDestroy(void* e) { (void)e; return 0; }
int hipEventRecord(void* e, void* s) { (void)e, (void)s; return 0; }
int hipEventSynchronize(void* e) { (void)e; return 0; }
/* every measured time is shorter than the one before */
int hipEventElapsedTime(float* ms, void* a, void* b) {
  (void)a, (void)b;
  *ms = 1000.0f / (float)++elapsed_calls;
  return 0;
}
