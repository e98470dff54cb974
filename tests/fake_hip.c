/* A HIP runtime without a device, for tests of the library's host code: memory is the host's and zeroed, copies
 * happen at once, kernels are noted by name and not run.  Loaded with global visibility before libapss.so, whose
 * calls then end here; a hook may stand in for the kernels.  As in ROCm 7, hipGetLastError gives the last failure and successful calls do not clear it.
 */
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>

#define MAX_FUNCS 512
#define MAX_LAUNCHES 4096

static hipError_t last;
static hipError_t fail(hipError_t e) { last = e; return e; }

static const void* func_at[MAX_FUNCS];
static const char* func_name[MAX_FUNCS];
static int nfuncs;
static const char* launched[MAX_LAUNCHES];
static int nlaunched;

static long mallocs, malloc_from, malloc_times;
static long events, event_from, event_times;
static long live;
static void (*hook)(const char* kernel, void** args);

/* allocations (events) from the k-th from now on fail, that many of them */
void fake_fail_mallocs(long k, long times) { mallocs = 0; malloc_from = k; malloc_times = times; }
void fake_fail_events(long k, long times) { events = 0; event_from = k; event_times = times; }
long fake_mallocs(void) { return mallocs; }
long fake_live(void) { return live; }
void fake_forget_launches(void) { nlaunched = 0; }
int fake_launches(void) { return nlaunched; }
const char* fake_launch(int k) { return launched[k]; }
/* called in place of every kernel */
void fake_hook(void (*f)(const char*, void**)) { hook = f; }

hipError_t hipMalloc(void** p, size_t size) {
  const long k = mallocs++;
  if (malloc_times > 0 && k >= malloc_from && k < malloc_from + malloc_times) return fail(hipErrorOutOfMemory);
  *p = calloc(size ? size : 1, 1);
  if (!*p) return fail(hipErrorOutOfMemory);
  ++live;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (p) --live;
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t size, unsigned int flags) {
  (void)flags;
  *p = calloc(size ? size : 1, 1);
  return *p ? hipSuccess : fail(hipErrorOutOfMemory);
}
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind kind, hipStream_t s) {
  (void)kind; (void)s;
  if (n && (!dst || !src)) return fail(hipErrorInvalidValue);
  if (n) memmove(dst, src, n);
  return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void* dst, size_t dp, const void* src, size_t sp, size_t w, size_t h, hipMemcpyKind kind,
                            hipStream_t s) {
  (void)kind; (void)s;
  for (size_t k = 0; k < h; ++k) memmove((char*)dst + k * dp, (const char*)src + k * sp, w);
  return hipSuccess;
}
hipError_t hipGetLastError(void) {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t e) {
  return e == hipSuccess ? "no error" : e == hipErrorOutOfMemory ? "out of memory" : e == hipErrorInvalidValue ? "invalid argument" : "error";
}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int d) { return d ? fail(hipErrorInvalidDevice) : hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int d) {
  (void)a; (void)d;
  *v = 256;
  return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int d) {
  (void)d;
  memset(p, 0, sizeof(*p));
  p->totalGlobalMem = 288ull << 30;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int threads, size_t lds) {
  (void)f; (void)threads; (void)lds;
  *n = 2;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void* symbol) {
  static void* mem;
  (void)symbol;
  if (!mem) mem = calloc(128, 1 << 20);
  *p = mem;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned flags) {
  (void)flags;
  *e = (hipEvent_t)malloc(1);
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  const long k = events++;
  (void)e; (void)s;
  if (event_times > 0 && k >= event_from && k < event_from + event_times) return fail(hipErrorUnknown);
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
  (void)a; (void)b;
  *ms = 0.0f;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned int flags) {
  (void)flags;
  *s = (hipStream_t)malloc(1);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { free(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { (void)s; return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode m) { (void)s; (void)m; return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) { (void)s; *g = (hipGraph_t)malloc(1); return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t g) { free(g); return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t* node, char* log, size_t n) {
  (void)g; (void)node; (void)log; (void)n;
  *x = (hipGraphExec_t)malloc(1);
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t s) { (void)x; (void)s; return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) { free(x); return hipSuccess; }

static __thread dim3 cfg_grid, cfg_block;
static __thread size_t cfg_lds;
static __thread hipStream_t cfg_stream;

hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
  cfg_grid = grid;
  cfg_block = block;
  cfg_lds = lds;
  cfg_stream = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
  *grid = cfg_grid;
  *block = cfg_block;
  *lds = cfg_lds;
  *s = cfg_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t s) {
  (void)lds; (void)s;
  if (!grid.x || !block.x) return fail(hipErrorInvalidValue);
  for (int k = 0; k < nfuncs; ++k) {
    if (func_at[k] != f) continue;
    if (nlaunched < MAX_LAUNCHES) launched[nlaunched++] = func_name[k];
    if (hook) hook(func_name[k], args);
  }
  return hipSuccess;
}

void** __hipRegisterFatBinary(const void* data) {
  static void* module;
  (void)data;
  return &module;
}
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* f, char* device_function, const char* name, unsigned int limit,
                           void* tid, void* bid, dim3* block, dim3* grid, int* warp) {
  (void)m; (void)device_function; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)warp;
  if (nfuncs < MAX_FUNCS) {
    func_at[nfuncs] = f;
    func_name[nfuncs++] = name;
  }
}
void __hipRegisterVar(void** m, void* var, char* host, char* name, int ext, size_t size, int constant, int global) {
  (void)m; (void)var; (void)host; (void)name; (void)ext; (void)size; (void)constant; (void)global;
}
