// Cache of idle device blocks behind ScratchBuf: one list per device, oldest first.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <new>
#include <vector>

#include "common.hpp"

namespace aqt {
namespace {

struct Block {
  void* p;
  size_t bytes;
};
constexpr int kMaxDevices = 64;
struct DeviceCache {
  std::vector<Block> idle;   // in the order they came back
  size_t total = 0;
  int contexts = 0;
};
std::mutex g_mutex;

// The device's cache; null if there is none (device index, no host memory for it): blocks are
// then allocated and freed as they come and go.
DeviceCache* cache_of(int device) {
  static DeviceCache* c = new (std::nothrow) DeviceCache[kMaxDevices];   // outlives every static destructor
  return (c && device >= 0 && device < kMaxDevices) ? c + device : nullptr;
}

// Frees the oldest blocks until at most `limit` bytes are cached (the mutex is held).
void trim(DeviceCache& c, size_t limit) {
  size_t k = 0;
  while (k < c.idle.size() && c.total > limit) {
    c.total -= c.idle[k].bytes;
    (void)hipFree(c.idle[k].p);
    ++k;
  }
  c.idle.erase(c.idle.begin(), c.idle.begin() + static_cast<std::ptrdiff_t>(k));
}

}  // namespace

hipError_t scratch_get(int device, size_t n, void** p, size_t* bytes) {
  n = std::max<size_t>((n + 255) & ~size_t(255), 256);
  if (DeviceCache* own = cache_of(device)) {
    std::lock_guard<std::mutex> lock(g_mutex);
    DeviceCache& c = *own;
    size_t best = c.idle.size();
    for (size_t k = 0; k < c.idle.size(); ++k)
      if (c.idle[k].bytes >= n && c.idle[k].bytes <= 2 * n &&
          (best == c.idle.size() || c.idle[k].bytes < c.idle[best].bytes))
        best = k;
    if (best < c.idle.size()) {
      *p = c.idle[best].p;
      *bytes = c.idle[best].bytes;
      c.total -= c.idle[best].bytes;
      c.idle.erase(c.idle.begin() + static_cast<std::ptrdiff_t>(best));
      return hipSuccess;
    }
  }
  hipError_t e = hipMalloc(p, n);
  if (e == hipErrorOutOfMemory) {
    (void)hipGetLastError();
    scratch_flush();
    e = hipMalloc(p, n);
  }
  if (e == hipSuccess) *bytes = n;
  return e;
}

void scratch_put(int device, void* p, size_t bytes) {
  DeviceCache* own = cache_of(device);
  if (own && bytes <= kScratchCacheBytes) {
    std::lock_guard<std::mutex> lock(g_mutex);
    DeviceCache& c = *own;
    try {
      c.idle.push_back(Block{p, bytes});
      c.total += bytes;
      trim(c, kScratchCacheBytes);
      return;
    } catch (...) {   // no host memory for the list: free the block instead
    }
  }
  (void)hipFree(p);
}

void scratch_flush() {
  std::lock_guard<std::mutex> lock(g_mutex);
  for (int d = 0; d < kMaxDevices; ++d)
    if (DeviceCache* c = cache_of(d)) trim(*c, 0);
}

void scratch_release(int device) {
  DeviceCache* c = cache_of(device);
  if (!c) return;
  std::lock_guard<std::mutex> lock(g_mutex);
  trim(*c, 0);
}

void scratch_context(int device, int delta) {
  DeviceCache* c = cache_of(device);
  if (!c) return;
  std::lock_guard<std::mutex> lock(g_mutex);
  c->contexts += delta;
  if (c->contexts <= 0) trim(*c, 0);
}

}  // namespace aqt
