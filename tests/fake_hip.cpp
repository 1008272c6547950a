// A HIP runtime of memory and bookkeeping alone, for tests of the library's
// host path without a GPU: loaded with RTLD_GLOBAL before libromap.so, its
// functions take the place of the runtime's.  Kernels do not run; their
// launches are counted, checked against the limits that the runtime has, and
// the arguments of some inspected.  "Device" memory is zeroed host memory that
// takes room only where it is written.
//
// fake_* functions set a condition or read what was seen.
#include <sys/mman.h>

#include <cstring>
#include <map>
#include <string>

#include "romap_device.h"

namespace {

struct FakeStream { int busy = 0; };  // graph launches not yet waited for
struct FakeExec { FakeStream* busy_on = nullptr; };

bool g_capturing = false;   // a caller captures the contexts' streams
bool g_own_capture = false; // the library captures
int g_fail_host = 0;
int64_t g_launches = 0, g_busy_destroyed = 0, g_graph_launches = 0, g_max_slots = 0;
std::map<void*, size_t> g_size;
std::map<const void*, std::string> g_kernel;
std::map<std::string, int64_t> g_threads;  // work-items launched, by kernel
dim3 g_grid, g_block;
size_t g_shm;
hipStream_t g_stream;

hipError_t alloc(void** p, size_t n) {
  n = n ? n : 1;
  *p = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (*p == MAP_FAILED) return hipErrorOutOfMemory;
  g_size[*p] = n;
  return hipSuccess;
}

hipError_t release(void* p) {
  auto it = g_size.find(p);
  if (p && it == g_size.end()) return hipErrorInvalidValue;
  if (p) {
    munmap(p, it->second);
    g_size.erase(it);
  }
  return hipSuccess;
}

}  // namespace

extern "C" {

// ---- conditions and observations
void fake_capture(int on) { g_capturing = on; }
void fake_fail_host_malloc(int n) { g_fail_host = n; }
int64_t fake_launches() { return g_launches; }
int64_t fake_graph_launches() { return g_graph_launches; }
int64_t fake_busy_graphs_destroyed() { return g_busy_destroyed; }
int64_t fake_max_record_slots() { return g_max_slots; }
int64_t fake_threads(const char* kernel) {
  int64_t n = 0;
  for (auto& k : g_threads)
    if (k.first.find(kernel) != std::string::npos) n += k.second;
  return n;
}

// ---- module registration and launches
void** __hipRegisterFatBinary(const void*) {
  static void* module;
  return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*,
                           void*, void*, int*) {
  g_kernel[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shm, hipStream_t st) {
  g_grid = grid, g_block = block, g_shm = shm, g_stream = st;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shm, hipStream_t* st) {
  *grid = g_grid, *block = g_block, *shm = g_shm, *st = g_stream;
  return hipSuccess;
}
static hipError_t g_last = hipSuccess;
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, hipStream_t) {
  // the runtime's limit: fewer than 2^32 work-items in x
  if ((uint64_t)grid.x * block.x >= (uint64_t(1) << 32) || grid.x == 0)
    return g_last = hipErrorInvalidConfiguration;
  ++g_launches;
  const std::string& name = g_kernel[f];
  g_threads[name] += (int64_t)grid.x * grid.y * block.x;
  if (name.find("k_bin_scatter") != std::string::npos) {
    const StepArgs& a = *(const StepArgs*)args[0];
    for (int i = 0; i < a.n_bpairs; ++i) {
      const int64_t n = (int64_t)a.bpairs[i].R * a.bpairs[i].cap;
      g_max_slots = n > g_max_slots ? n : g_max_slots;
    }
  }
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = g_last;
  g_last = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t) { return "fake HIP error"; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { return alloc(p, size_t(64) << 20); }

// ---- memory
hipError_t hipMalloc(void** p, size_t n) { return alloc(p, n); }
hipError_t hipFree(void* p) { return release(p); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  if (g_fail_host > 0) {
    --g_fail_host;
    return hipErrorOutOfMemory;
  }
  return alloc(p, n);
}
hipError_t hipHostFree(void* p) { return release(p); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  return std::memcpy(d, s, n), hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  return std::memcpy(d, s, n), hipSuccess;
}
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }  // it is zero

// ---- streams and events
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = (hipStream_t) new FakeStream;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { return delete (FakeStream*)s, hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
  if (g_capturing) return hipErrorStreamCaptureUnsupported;
  if (s) ((FakeStream*)s)->busy = 0;
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* st) {
  *st = g_capturing || g_own_capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return *e = (hipEvent_t) new int, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { return delete (int*)e, hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 0.1f, hipSuccess; }

// ---- graphs
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
  return g_own_capture = true, hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  g_own_capture = false;
  return *g = (hipGraph_t) new int, hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  return *e = (hipGraphExec_t) new FakeExec, hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { return delete (int*)g, hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t s) {
  ((FakeExec*)e)->busy_on = (FakeStream*)s;
  ((FakeStream*)s)->busy = 1;
  ++g_graph_launches;
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
  FakeExec* x = (FakeExec*)e;
  g_busy_destroyed += x->busy_on && x->busy_on->busy;
  return delete x, hipSuccess;
}

}  // extern "C"
