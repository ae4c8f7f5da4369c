/* Stands in for the HIP runtime in CPU tests of the library's host side: the calls the library makes are
 * reported to two callbacks, which decide what they return; nothing runs.  Loaded before the library, it
 * serves the library's references by its soname (libamdhip64.so.7). */
#define __HIP_PLATFORM_AMD__
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>

typedef int (*launch_fn)(const char* kernel, unsigned grid, unsigned block, unsigned lds, void* stream, void** args,
                         void* start, void* stop);
typedef int (*call_fn)(const char* name, void* subject);
static launch_fn on_launch;
static call_fn on_call;
void stub_callbacks(launch_fn l, call_fn c) { on_launch = l; on_call = c; }
static int call(const char* name, const void* subject) { return on_call ? on_call(name, (void*)subject) : 0; }

/* what the library registers when it is loaded */
static struct { const void* function; const char* name; } kernels[4096];
static int n_kernels;
static struct { const void* variable; size_t size; void* at; } variables[64];
static int n_variables;
void** __hipRegisterFatBinary(const void* data) { static void* module; (void)data; return &module; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* function, char* device, const char* name, unsigned limit, void* tid, void* bid,
                           void* bd, void* gd, int* ws) {
  (void)m; (void)device; (void)limit; (void)tid; (void)bid; (void)bd; (void)gd; (void)ws;
  if (n_kernels < 4096) { kernels[n_kernels].function = function; kernels[n_kernels++].name = name; }
}
void __hipRegisterVar(void** m, void* variable, char* host, char* device, int ext, size_t size, int constant, int global) {
  (void)m; (void)host; (void)device; (void)ext; (void)constant; (void)global;
  if (n_variables < 64) { variables[n_variables].variable = variable; variables[n_variables++].size = size; }
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* l, hipStream_t* s) { (void)g; (void)b; (void)l; (void)s; return hipErrorUnknown; }

static hipError_t launch(const void* f, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t s, hipEvent_t t0, hipEvent_t t1) {
  const char* name = "?";
  for (int i = 0; i < n_kernels; ++i) if (kernels[i].function == f) name = kernels[i].name;
  /* the runtime's own limit on a launch: threads in all are a 32-bit number */
  if ((unsigned long long)grid.x * block.x > 0xFFFFFFFFull) return hipErrorInvalidConfiguration;
  return (hipError_t)(on_launch ? on_launch(name, grid.x, block.x, (unsigned)lds, s, args, t0, t1) : 0);
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t lds, hipStream_t s) { return launch(f, g, b, args, lds, s, 0, 0); }
hipError_t hipExtLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t lds, hipStream_t s, hipEvent_t t0, hipEvent_t t1, int flags) {
  (void)flags;
  return launch(f, g, b, args, lds, s, t0, t1);
}

hipError_t hipGetDevice(int* d) { *d = 0; return (hipError_t)call("hipGetDevice", 0); }
const char* hipGetErrorName(hipError_t e) { return e == hipErrorInvalidConfiguration ? "hipErrorInvalidConfiguration" : "some error"; }
const char* hipGetErrorString(hipError_t e) { (void)e; return "as the test asked"; }
hipError_t hipGetLastError(void) { return (hipError_t)call("hipGetLastError", 0); }
/* the callback says whether the stream is being captured (1) or cannot be asked (negative) */
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  const int r = call("hipStreamIsCapturing", s);
  *st = r == 1 ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return r < 0 ? hipErrorInvalidValue : hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) { (void)m; return (hipError_t)call("hipThreadExchangeStreamCaptureMode", 0); }
/* the callback says what the memory is: 0 device, 1 host, negative = not known to the runtime */
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  const int r = call("hipPointerGetAttributes", p);
  memset(a, 0, sizeof(*a));
  a->type = r == 1 ? hipMemoryTypeHost : hipMemoryTypeDevice;
  return r < 0 ? hipErrorInvalidValue : hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { *p = calloc(1, n); return (hipError_t)call("hipMalloc", (void*)n); }
hipError_t hipFree(void* p) { free(p); return (hipError_t)call("hipFree", 0); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned f) { (void)f; *p = calloc(1, n); return (hipError_t)call("hipHostMalloc", (void*)n); }
hipError_t hipHostFree(void* p) { free(p); return (hipError_t)call("hipHostFree", 0); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k) { (void)k; memcpy(d, s, n); return (hipError_t)call("hipMemcpy", (void*)n); }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t st) { (void)k; (void)st; memcpy(d, s, n); return (hipError_t)call("hipMemcpyAsync", (void*)n); }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t st) { (void)st; memset(d, v, n); return (hipError_t)call("hipMemsetAsync", (void*)n); }
hipError_t hipGetSymbolAddress(void** at, const void* symbol) {
  for (int i = 0; i < n_variables; ++i) if (variables[i].variable == symbol) {
    if (!variables[i].at) variables[i].at = calloc(1, variables[i].size);
    *at = variables[i].at;
    return (hipError_t)call("hipGetSymbolAddress", 0);
  }
  return hipErrorInvalidSymbol;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned f) { (void)f; *s = (hipStream_t)malloc(1); return (hipError_t)call("hipStreamCreateWithFlags", 0); }
hipError_t hipStreamDestroy(hipStream_t s) { free(s); return (hipError_t)call("hipStreamDestroy", 0); }
hipError_t hipStreamSynchronize(hipStream_t s) { return (hipError_t)call("hipStreamSynchronize", s); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned f) { (void)f; *e = (hipEvent_t)malloc(1); return (hipError_t)call("hipEventCreateWithFlags", 0); }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return (hipError_t)call("hipEventDestroy", 0); }
hipError_t hipEventQuery(hipEvent_t e) { return (hipError_t)call("hipEventQuery", e); }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { (void)s; return (hipError_t)call("hipEventRecord", e); }
hipError_t hipEventSynchronize(hipEvent_t e) { return (hipError_t)call("hipEventSynchronize", e); }
