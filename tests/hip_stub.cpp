// The HIP runtime calls that libqsv makes, as a host-only recorder: memory is
// host memory, copies are done at once, kernels are counted and not run. It lets
// tests look at the host runtime (what is allocated, captured, replayed, waited
// for) and make single calls fail, on a machine without a GPU. Loaded with
// RTLD_GLOBAL before libqsv, whose HIP symbols it then provides.
//
// Freed blocks are never handed out again, so that an address names one
// allocation.
#include <hip/hip_runtime_api.h>

#include <sys/mman.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <vector>

namespace {
std::mutex mu;
struct Config {
  dim3 grid, block;
  size_t lds;
  hipStream_t st;
};
thread_local std::vector<Config> configs;
std::map<const void*, std::string> names;
std::map<std::string, long> counts;            // calls by name ("kernel <mangled name>" for launches)
std::set<void*> live;                          // device blocks
std::map<void*, std::set<void*>> graph_blocks; // per graph: the device blocks live when it was captured
std::string fail_name;                         // the call that fails
long fail_skip = -1;                           // after this many more successes
long stale = 0;                                // replays of graphs of which a block has been freed since
long pending = 0;                              // asynchronous work since the last wait
std::string grid_name;                         // the kernel whose workgroups are added up
std::vector<long> grids;                       // of each launch of it

void count(const char* n) { ++counts[n]; }
// counts a call of n; true: it has to fail
bool call(const char* n) {
  count(n);
  if (fail_skip < 0 || fail_name != n) return false;
  return fail_skip-- == 0;
}
template <class T>
T handle() {
  return reinterpret_cast<T>(std::malloc(16));
}
}  // namespace

#define GUARD std::lock_guard<std::mutex> lk(mu)

extern "C" {
// the recorder's own entry points
long stub_count(const char* n) {
  GUARD;
  long c = 0;
  for (const auto& e : counts)
    if (e.first.find(n) != std::string::npos) c += e.second;
  return c;
}
void stub_fail(const char* n, long skip) {
  GUARD;
  fail_name = n;
  fail_skip = skip;
}
long stub_stale_replays() { return stale; }
long stub_pending() { return pending; }
// from here on, the workgroups of the launches of the kernel whose name holds n
void stub_watch(const char* n) {
  GUARD;
  grid_name = n;
  grids.clear();
}
long stub_grid(long i) {
  GUARD;
  return i < (long)grids.size() ? grids[i] : -1;
}

// the HIP runtime
void** __hipRegisterFatBinary(const void*) { return handle<void**>(); }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*,
                           int*) {
  GUARD;
  names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t st) {
  configs.push_back({g, b, lds, st});
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* st) {
  const Config c = configs.back();
  configs.pop_back();
  *g = c.grid;
  *b = c.block;
  *lds = c.lds;
  *st = c.st;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3, void**, size_t, hipStream_t) {
  GUARD;
  ++counts["kernel " + names[f]];
  if (!grid_name.empty() && names[f].find(grid_name) != std::string::npos) grids.push_back((long)g.x);
  ++pending;
  return hipSuccess;
}
hipError_t hipGetDeviceCount(int* n) { return *n = 1, hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  std::memset(p, 0, sizeof(*p));
  std::strcpy(p->gcnArchName, "gfx950");
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 160 << 10;
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* fr, size_t* tot) { return *fr = *tot = (size_t)4 << 30, hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "an error of the recorder"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) {
  GUARD;
  count("hipFuncSetAttribute");
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  GUARD;
  count("hipOccupancy");
  return *n = 2, hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static void* const block = std::malloc((size_t)64 << 20);
  return *p = block, hipSuccess;
}
// (device memory holds different words, so that no two shots look alike)
hipError_t hipMalloc(void** p, size_t n) {
  GUARD;
  if (call("hipMalloc")) return hipErrorOutOfMemory;
  // (address space only; the pages that are written become memory)
  void* m = mmap(nullptr, n + 8, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (m == MAP_FAILED) return hipErrorOutOfMemory;
  uint64_t* w = static_cast<uint64_t*>(m);
  for (size_t i = 0; i < n / 8 && i < ((size_t)1 << 17); ++i) w[i] = i;
  live.insert(w);
  return *p = w, hipSuccess;
}
hipError_t hipFree(void* p) {
  GUARD;
  count("hipFree");
  live.erase(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  GUARD;
  if (call("hipHostMalloc")) return hipErrorOutOfMemory;
  return *p = std::malloc(n), hipSuccess;
}
hipError_t hipHostFree(void* p) {
  GUARD;
  count("hipHostFree");
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { return std::memmove(d, s, n), hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  GUARD;
  if (call("hipMemcpyAsync")) return hipErrorUnknown;
  ++pending;
  std::memmove(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  GUARD;
  ++pending;
  std::memset(d, v, n);
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return *s = handle<hipStream_t>(), hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) {
  GUARD;
  count("hipStreamSynchronize");
  pending = 0;
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
  GUARD;
  if (call("hipEventCreate")) return hipErrorOutOfMemory;
  return *e = handle<hipEvent_t>(), hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  GUARD;
  count(e ? "hipEventRecord" : "record of no event");
  return e ? hipSuccess : hipErrorInvalidHandle;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 1.f, hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
  GUARD;
  count("hipStreamBeginCapture");
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  GUARD;
  *g = handle<hipGraph_t>();
  graph_blocks[*g] = live;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
  GUARD;
  *e = handle<hipGraphExec_t>();
  graph_blocks[*e] = graph_blocks[g];
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t) {
  GUARD;
  count("hipGraphLaunch");
  ++pending;
  for (void* b : graph_blocks[e])
    if (!live.count(b)) {
      ++stale;
      break;
    }
  return hipSuccess;
}
}
