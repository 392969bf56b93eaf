// A HIP runtime without a device, for tests of the library's host side: memory is host
// memory, copies are copies, and a kernel launch runs nothing but is logged by its kernel's
// name (graph replays too). Loaded before libfe.so with its symbols global, it takes the
// place of the real runtime there. sweep_finish and vec_finish, whose results the host
// reads, write recognisable values.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <vector>

namespace {

struct Launch {
  std::string name;
  dim3 grid, block;
};
struct Graph {
  std::vector<Launch> nodes;
};

std::map<const void*, std::string> g_names;
std::vector<Launch> g_log;
std::map<hipStream_t, Graph*> g_capturing;
std::set<void*> g_host;                 // live pinned allocations
long g_host_allocs = 0;
bool g_host_full = false;
int g_slots = 2;
void* g_energy = nullptr;               // where the last sweep_finish wrote, and how many
unsigned g_energies = 0;
double g_next = 1.0;                    // its first value (the others follow by 1)
std::vector<Launch> g_calls;            // pushed call configurations
std::vector<size_t> g_shared;
std::vector<hipStream_t> g_streams;
std::mutex g_mu;

}  // namespace

extern "C" {

// ---- what the tests read and set ----
long stub_log_size() { return (long)g_log.size(); }
const char* stub_log_name(long i) { return g_log[i].name.c_str(); }
unsigned stub_log_blocks(long i) { return g_log[i].grid.x; }
void stub_log_clear() { g_log.clear(); }
long stub_host_allocs() { return g_host_allocs; }
long stub_host_live() { return (long)g_host.size(); }
void stub_host_full(int full) { g_host_full = full != 0; }
void stub_slots(int slots) { g_slots = slots; }
void* stub_energy() { return g_energy; }
unsigned stub_energies() { return g_energies; }
void stub_next(double v) { g_next = v; }

// ---- code objects and launches ----
void** __hipRegisterFatBinary(const void*) {
  static void* handle = nullptr;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*,
                           int*) {
  g_names[host] = device;
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}

hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream) {
  g_calls.push_back(Launch{"", grid, block});
  g_shared.push_back(shared);
  g_streams.push_back(stream);
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream) {
  *grid = g_calls.back().grid;
  *block = g_calls.back().block;
  *shared = g_shared.back();
  *stream = g_streams.back();
  g_calls.pop_back();
  g_shared.pop_back();
  g_streams.pop_back();
  return hipSuccess;
}

hipError_t hipLaunchKernel(const void* host, dim3 grid, dim3 block, void** args, size_t, hipStream_t stream) {
  const Launch l{g_names.at(host), grid, block};
  const auto it = g_capturing.find(stream);
  if (it != g_capturing.end()) {
    it->second->nodes.push_back(l);
    return hipSuccess;
  }
  g_log.push_back(l);
  if (l.name.find("sweep_finish") != std::string::npos) {
    g_energy = *static_cast<void**>(args[2]);
    g_energies = grid.x;
    for (unsigned b = 0; g_energy && b < grid.x; ++b) static_cast<double*>(g_energy)[b] = g_next + b;
  } else if (l.name.find("vec_finish") != std::string::npos) {
    for (unsigned k = 0; k < grid.x; ++k) (*static_cast<double**>(args[1]))[k] = 0.25;
  }
  return hipSuccess;
}

hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = g_slots;
  return hipSuccess;
}

// ---- memory ----
hipError_t hipMalloc(void** p, size_t n) {
  *p = std::calloc(n ? n : 1, 1);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  std::lock_guard<std::mutex> lock(g_mu);
  if (g_host_full) return hipErrorOutOfMemory;
  *p = std::calloc(n, 1);
  g_host.insert(*p);
  ++g_host_allocs;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  std::lock_guard<std::mutex> lock(g_mu);
  if (!g_host.erase(p)) return hipErrorInvalidValue;
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(dst, src, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* dst, int v, size_t n, hipStream_t) {
  std::memset(dst, v, n);
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static void* scratch = std::calloc(1 << 20, 1);
  *p = scratch;
  return hipSuccess;
}

// ---- device, streams, events, errors ----
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
  std::memset(p, 0, sizeof(*p));
  std::strcpy(p->gcnArchName, "stub");
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = reinterpret_cast<hipStream_t>(std::malloc(1));
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  std::free(s);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = reinterpret_cast<hipEvent_t>(std::malloc(1));
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
  std::free(e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub error"; }

// ---- graphs ----
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  g_capturing[s] = new Graph;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) {
  *g = reinterpret_cast<hipGraph_t>(g_capturing.at(s));
  g_capturing.erase(s);
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
  *e = reinterpret_cast<hipGraphExec_t>(new Graph(*reinterpret_cast<Graph*>(g)));
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
  delete reinterpret_cast<Graph*>(g);
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
  delete reinterpret_cast<Graph*>(e);
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t) {
  const Graph* g = reinterpret_cast<const Graph*>(e);
  g_log.insert(g_log.end(), g->nodes.begin(), g->nodes.end());
  return hipSuccess;
}

}  // extern "C"
