#include "hip_stub.hpp"

#include <cstring>
#include <mutex>
#include <new>

namespace stub {
size_t host_allocations = ~size_t(0);
std::map<char*, size_t> live;
size_t used = 0, limit = size_t(288) << 30, peak = 0;
size_t allocations = ~size_t(0);
std::vector<Call> calls;
std::function<void(const Call&)> on_call;
std::function<void(void*, const void*, size_t)> on_download;

namespace {
char* next_block = reinterpret_cast<char*>(size_t(1) << 44);
std::map<const void*, std::string>& kernels() {
  static std::map<const void*, std::string> m;
  return m;
}
// The stub's own bookkeeping is one thread's at a time and is not counted.
std::recursive_mutex lock;
struct Uncounted {
  std::lock_guard<std::recursive_mutex> own{lock};
  size_t n = host_allocations;
  Uncounted() { host_allocations = ~size_t(0); }
  ~Uncounted() { host_allocations = n; }
};
struct Config {
  dim3 grid, block;
  size_t shared;
  hipStream_t stream;
} config;
void note(Call c) {
  std::lock_guard<std::recursive_mutex> own(lock);
  if (on_call) on_call(c);
  c.args = nullptr;
  calls.push_back(c);
}
void note(const char* name, hipStream_t s = nullptr) {
  Uncounted u;
  note(Call{name, s, dim3(1), nullptr});
}
bool on_device(const void* p) {
  const char* c = static_cast<const char*>(p);
  auto it = live.upper_bound(const_cast<char*>(c));
  if (it == live.begin()) return false;
  --it;
  return c < it->first + it->second;
}
void copy(void* dst, const void* src, size_t n) {
  if (!on_device(dst)) {
    std::memset(dst, 0, n);
    if (on_download) on_download(dst, src, n);
  }
}
}  // namespace
}  // namespace stub

using namespace stub;

void* operator new(size_t n) {
  if (!host_allocations) throw std::bad_alloc();
  if (host_allocations != ~size_t(0)) --host_allocations;
  if (void* p = std::malloc(n)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  Uncounted u;
  if (n > limit - used || !allocations) return hipErrorOutOfMemory;
  --allocations;
  live[next_block] = n;
  *p = next_block;
  next_block += (n + 4096) & ~size_t(4095);
  used += n;
  if (used > peak) peak = used;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (!p) return hipSuccess;
  Uncounted u;
  const auto it = live.find(static_cast<char*>(p));
  CHECK(it != live.end());
  used -= it->second;
  live.erase(it);
  note("hipFree");
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
  note("hipMemcpyAsync", st);
  copy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  note("hipMemcpy");
  copy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t st) {
  note("hipMemsetAsync", st);
  return hipSuccess;
}
hipError_t hipMemset(void*, int, size_t) {
  note("hipMemset");
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  note("hipStreamSynchronize", s);
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
  note("hipDeviceSynchronize");
  return hipSuccess;
}
hipError_t hipGetDeviceCount(int* n) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  std::memset(p, 0, sizeof(*p));
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  *p = next_block;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = reinterpret_cast<hipEvent_t>(8);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.f;
  return hipSuccess;
}
hipError_t hipStreamCreate(hipStream_t* s) {
  static size_t n = 0x1000;
  *s = reinterpret_cast<hipStream_t>(n += 16);
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return hipStreamCreate(s); }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t, hipStream_t s) {
  note(Call{kernels()[f], s, grid, args});
  return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t s) {
  config = Config{grid, block, shared, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* s) {
  *grid = config.grid;
  *block = config.block;
  *shared = config.shared;
  *s = config.stream;
  return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) {
  static void* h[1];
  return h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  kernels()[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
}
