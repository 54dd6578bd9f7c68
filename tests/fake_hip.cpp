// A stand-in for the HIP runtime, linked with the library's own objects so
// that the host side of the C ABI runs without a GPU: memory is host memory,
// copies are made, kernels are recorded and not run. Tests set limits and
// failures by name (fake_set), and read counts (fake_get) and the launches
// (fake_launch). One thread at a time.
#include <cxxabi.h>
#include <hip/hip_runtime_api.h>
#include <sys/mman.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

struct ihipStream_t {
  int device;
  bool capturing;
};
struct ihipEvent_t {};
struct ihipGraph {
  int launches;
};
struct hipGraphExec {
  int launches;
};

namespace {

struct Launch {
  std::string name;
  long long v[9];  // grid, block, stream's device, current device, captured
};

std::map<std::string, long long> vars;
std::map<const void*, std::string> kernels;
std::map<void*, size_t> blocks;
std::vector<Launch> launches;
hipError_t last = hipSuccess;
int current = 0, captured = 0;
hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;

long long& var(const char* k) { return vars[k]; }

hipError_t give(hipError_t e) {
  if (e != hipSuccess) last = e;
  return e;
}

// True once the call counted under `counter` is the one that `fail` names.
bool due(const char* counter, const char* fail) {
  return ++var(counter) == var(fail);
}

// Calls that another capture of this thread forbids outside relaxed mode
// ("thread_captures": the caller is recording on a stream of its own).
bool forbidden() {
  if (!var("thread_captures") || mode == hipStreamCaptureModeRelaxed) return false;
  var("captures_broken") += 1;
  return true;
}

}  // namespace

extern "C" {

// ---- controls -------------------------------------------------------------
void fake_reset() {
  vars.clear();
  launches.clear();
  last = hipSuccess;
  current = 0;
  mode = hipStreamCaptureModeGlobal;
}
void fake_set(const char* k, long long v) { var(k) = v; }
long long fake_get(const char* k) {
  const std::string s(k);
  if (s == "launches") return (long long)launches.size();
  if (s == "current") return current;
  return var(k);
}
int fake_launch(int i, char* name, int size, long long* v) {
  const Launch& l = launches.at(i);
  std::strncpy(name, l.name.c_str(), size - 1);
  name[size - 1] = 0;
  std::memcpy(v, l.v, sizeof(l.v));
  return 0;
}
int fake_kernel_count() { return (int)kernels.size(); }
void fake_kernel_name(int i, char* name, int size) {
  auto it = kernels.begin();
  std::advance(it, i);
  std::strncpy(name, it->second.c_str(), size - 1);
  name[size - 1] = 0;
}

// ---- registration and launch ------------------------------------------------
void** __hipRegisterFatBinary(const void*) {
  static void* module;
  return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name,
                           unsigned, void*, void*, void*, void*, int*) {
  int status = 1;
  char* d = abi::__cxa_demangle(name, nullptr, nullptr, &status);
  kernels[host] = status == 0 ? d : name;
  std::free(d);
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

static dim3 push_grid, push_block;
static size_t push_shared;
static hipStream_t push_stream;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t m, hipStream_t s) {
  push_grid = g;
  push_block = b;
  push_shared = m;
  push_stream = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* m, hipStream_t* s) {
  *g = push_grid;
  *b = push_block;
  *m = push_shared;
  *s = push_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void**, size_t,
                           hipStream_t s) {
  // documented limits: 1024 threads per workgroup, fewer than 2^32 threads
  // in each direction
  const auto over = [](unsigned n, unsigned t) {
    return (unsigned long long)n * t >> 32 != 0 || n == 0;
  };
  if (b.x * b.y * b.z > 1024 || over(g.x, b.x) || over(g.y, b.y) || over(g.z, b.z))
    return give(hipErrorInvalidConfiguration);
  if (due("kernel_calls", "fail_kernel")) return give(hipErrorUnknown);
  launches.push_back({kernels[f],
                      {g.x, g.y, g.z, b.x, b.y, b.z, s ? s->device : -1, current,
                       s && s->capturing}});
  if (s && s->capturing) ++captured;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int,
                                                        size_t) {
  if (var("fail_occupancy")) return give(hipErrorUnknown);
  *n = 2;
  return hipSuccess;
}

// ---- devices, errors ----------------------------------------------------------
hipError_t hipGetDevice(int* d) {
  *d = current;
  return hipSuccess;
}
hipError_t hipSetDevice(int d) {
  current = d;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 256;  // compute units, the only attribute asked for
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t) { return "error of the stand-in"; }

// ---- memory ---------------------------------------------------------------------
hipError_t hipMalloc(void** p, size_t n) {
  if (forbidden()) return give(hipErrorStreamCaptureUnsupported);
  const long long limit = var("memory");  // 0: no limit
  if (limit && var("allocated") + (long long)n > limit)
    return give(hipErrorOutOfMemory);
  *p = mmap(nullptr, n ? n : 1, PROT_READ | PROT_WRITE,
            MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (*p == MAP_FAILED) return give(hipErrorOutOfMemory);
  blocks[*p] = n ? n : 1;
  if (var("fill")) std::memset(*p, (int)var("fill"), n);
  var("allocated") += (long long)n;
  if (var("allocated") > var("peak")) var("peak") = var("allocated");
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  const auto it = blocks.find(p);
  if (it == blocks.end()) return give(hipErrorInvalidValue);
  var("allocated") -= (long long)it->second;
  munmap(p, it->second);
  blocks.erase(it);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind,
                          hipStream_t) {
  if (due("copies", "fail_copy")) return give(hipErrorUnknown);
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  if (v || var("fill")) std::memset(d, v, n);  // else it is zero already
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static char scratch[1 << 16];
  *p = scratch;
  return hipSuccess;
}

// ---- streams, events --------------------------------------------------------------
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  if (forbidden()) return give(hipErrorStreamCaptureUnsupported);
  *s = new ihipStream_t{current, false};
  var("streams") += 1;
  var(current ? "streams_on_1" : "streams_on_0") += 1;
  return hipSuccess;
}
hipError_t hipStreamCreate(hipStream_t* s) { return hipStreamCreateWithFlags(s, 0); }
hipError_t hipStreamDestroy(hipStream_t s) {
  delete s;
  var("streams") -= 1;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  if (forbidden()) return give(hipErrorStreamCaptureUnsupported);
  var("syncs") += 1;
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) {
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = new ihipEvent_t;
  var(current ? "events_on_1" : "events_on_0") += 1;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
  delete e;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}

// ---- capture ------------------------------------------------------------------------
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) {
  std::swap(*m, mode);
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  if (var("fail_is_capturing")) return give(hipErrorStreamCaptureImplicit);
  *st = s->capturing || var("stream_captures") ? hipStreamCaptureStatusActive
                                                : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  s->capturing = true;
  captured = 0;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) {
  s->capturing = false;
  *g = new ihipGraph{captured};
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t*,
                               char*, size_t) {
  if (due("instantiations", "fail_instantiate")) return give(hipErrorOutOfMemory);
  *x = new hipGraphExec{g->launches};
  var("graphs") += 1;
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
  delete g;
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x) {
  delete x;
  var("graphs") -= 1;
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t) {
  if (due("graph_calls", "fail_graph")) return give(hipErrorOutOfMemory);
  var("graph_kernels") += x->launches;
  return hipSuccess;
}

}  // extern "C"
