// A HIP runtime without a device, for host-side checks: memory is a range of addresses whose
// sizes are known, launches and waits are recorded in order, copies to the host give zeros
// unless the check answers them.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <functional>
#include <map>
#include <string>
#include <vector>

#define CHECK(cond)                                        \
  do {                                                     \
    if (!(cond)) {                                         \
      std::printf("%s:%d: %s\n", __FILE__, __LINE__, #cond); \
      std::exit(1);                                        \
    }                                                      \
  } while (0)

namespace stub {
struct Call {
  std::string name;           // kernel (mangled) or runtime call
  hipStream_t stream = nullptr;
  dim3 grid;
  void** args = nullptr;      // of a kernel, valid in on_call only
};
extern std::map<char*, size_t> live;          // allocated blocks
extern size_t used, limit, peak;              // bytes, the bytes there are, the most in use
extern size_t allocations;                    // on the device that still succeed
extern size_t host_allocations;               // operator new of the code under check, likewise
extern std::vector<Call> calls;               // in order
extern std::function<void(const Call&)> on_call;
extern std::function<void(void* dst, const void* src, size_t n)> on_download;
inline size_t count(const char* part) {
  size_t n = 0;
  for (const Call& c : calls) n += c.name.find(part) != std::string::npos;
  return n;
}
}  // namespace stub
