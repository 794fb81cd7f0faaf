// A stand-in for the HIP runtime on the CPU, for tests of the library's host
// code (fake_hip.py): device memory is host memory, copies happen at once,
// kernels do not run.  What the library asks of the runtime is recorded, and
// a test can set the conditions it reacts to: memory that runs out, a call
// that fails, another stream's capture or unfinished work.
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <map>
#include <mutex>
#include <string>

namespace {

std::recursive_mutex mu;
std::string log_;                        // one line per recorded call
std::map<char*, size_t> device, pinned;  // live allocations
std::map<const void*, std::string> kernels;
std::map<std::string, int> fail_at;  // call -> calls left before it fails
size_t limit = (size_t)288 << 30, used = 0;
bool fill = false;             // fresh device memory holds the doubles 0, 1, 2, ...
bool foreign_work = false;     // unfinished work on a stream that is not the library's
bool foreign_capture = false;  // such a stream is being captured (global mode)
thread_local hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
thread_local hipError_t last = hipSuccess;
dim3 cfg_grid, cfg_block;
size_t cfg_lds;
hipStream_t cfg_stream;

hipError_t rc(hipError_t e) { return last = e; }

bool fails(const char* call) {
  auto it = fail_at.find(call);
  return it != fail_at.end() && it->second-- == 0;
}

void note(const std::string& s) { log_ += s + "\n"; }

bool is_pinned(const void* p) {
  auto it = pinned.upper_bound((char*)p);
  return it != pinned.begin() && (--it, (char*)p < it->first + it->second);
}

}  // namespace

extern "C" {

// ------------------------------------------------------- the test's side
void fake_reset() { std::lock_guard<std::recursive_mutex> l(mu); log_.clear(); }
const char* fake_log() { return log_.c_str(); }
void fake_limit(size_t bytes) { limit = bytes; }
size_t fake_used() { return used; }
void fake_fill(int on) { fill = on; }
void fake_fail(const char* call, int after) { fail_at[call] = after; }
void fake_foreign_work(int on) { foreign_work = on; }
int fake_foreign_work_left() { return foreign_work; }
void fake_foreign_capture(int on) { foreign_capture = on; }
int fake_foreign_capture_left() { return foreign_capture; }

// ------------------------------------------------------------ the runtime
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof(*p));
  strcpy(p->gcnArchName, "gfx950");
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipGetLastError() { const hipError_t e = last; last = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t e) {
  static thread_local char s[32];
  snprintf(s, sizeof(s), "error %d", (int)e);
  return s;
}

// An allocation is unsafe while another stream's capture is under way, unless
// the thread has relaxed its mode: it fails and ends that capture.
static bool unsafe_now() {
  if (!foreign_capture || mode == hipStreamCaptureModeRelaxed) return false;
  foreign_capture = false;
  return true;
}
hipError_t hipMalloc(void** p, size_t n) {
  std::lock_guard<std::recursive_mutex> l(mu);
  note("malloc " + std::to_string(n));
  if (unsafe_now()) return rc(hipErrorStreamCaptureUnsupported);
  if (fails("malloc") || used + n > limit) return rc(hipErrorOutOfMemory);
  *p = calloc(n ? n : 1, 1);
  for (size_t i = 0; fill && i < n / 8; ++i) ((double*)*p)[i] = (double)i;
  device[(char*)*p] = n;
  used += n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  std::lock_guard<std::recursive_mutex> l(mu);
  if (!p) return hipSuccess;
  foreign_work = false;  // waits for the device
  note("free " + std::to_string(device[(char*)p]));
  used -= device[(char*)p];
  device.erase((char*)p);
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned int) {
  std::lock_guard<std::recursive_mutex> l(mu);
  note("hostmalloc " + std::to_string(n));
  if (unsafe_now()) return rc(hipErrorStreamCaptureUnsupported);
  if (fails("hostmalloc")) return rc(hipErrorOutOfMemory);
  *p = calloc(n, 1);
  pinned[(char*)*p] = n;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  std::lock_guard<std::recursive_mutex> l(mu);
  if (!pinned.erase((char*)p)) return rc(hipErrorInvalidValue);
  free(p);
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* free_b, size_t* total) {
  *free_b = limit - used;
  *total = limit;
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  std::lock_guard<std::recursive_mutex> l(mu);
  memset(a, 0, sizeof(*a));
  a->type = is_pinned(p) ? hipMemoryTypeHost : hipMemoryTypeUnregistered;
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) {
  std::lock_guard<std::recursive_mutex> l(mu);
  const void* host = k == hipMemcpyHostToDevice ? s : d;
  // the first words of what goes in, for a look at a batch's header
  std::string head;
  if (k == hipMemcpyHostToDevice && n >= 64)
    head = " " + std::to_string(((const int32_t*)s)[0]) + " " +
           std::to_string(((const int32_t*)s)[1]);
  note(std::string(k == hipMemcpyHostToDevice   ? "h2d "
                   : k == hipMemcpyDeviceToHost ? "d2h "
                                                : "d2d ") +
       std::to_string(n) + (is_pinned(host) ? " pinned" : " pageable") + head);
  if (fails("memcpy")) return rc(hipErrorUnknown);
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  memset(d, v, n);
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
  foreign_work = false;
  note("devicesync");
  return hipSuccess;
}

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned int) {
  *s = (hipStream_t)malloc(1);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { free((void*)s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { note("streamsync"); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned int) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) {
  std::swap(*m, mode);
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  *g = (hipGraph_t)malloc(1);
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  *e = (hipGraphExec_t)malloc(1);
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { note("graph"); return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t g) { free((void*)g); return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { free((void*)e); return hipSuccess; }
hipError_t hipLaunchHostFunc(hipStream_t, hipHostFn_t f, void* p) { f(p); return hipSuccess; }

hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  std::lock_guard<std::recursive_mutex> l(mu);
  if (fails("event")) return rc(hipErrorOutOfMemory);
  *e = (hipEvent_t)malloc(1);
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { free((void*)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  return e ? hipSuccess : rc(hipErrorInvalidHandle);
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  note("eventsync");
  return e ? hipSuccess : rc(hipErrorInvalidHandle);
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1; return hipSuccess; }

hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static void* a = calloc((size_t)256 << 20, 1);
  *p = a;
  return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned int,
                           void*, void*, dim3*, dim3*, int*) {
  kernels[host] = name;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
  cfg_grid = g, cfg_block = b, cfg_lds = lds, cfg_stream = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
  *g = cfg_grid, *b = cfg_block, *lds = cfg_lds, *s = cfg_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void**, size_t, hipStream_t) {
  std::lock_guard<std::recursive_mutex> l(mu);
  note("launch " + kernels[f] + " " + std::to_string(g.x) + "x" + std::to_string(b.x));
  return hipSuccess;
}

}  // extern "C"
