// Creating contexts while host allocations fail.  A process of its own: the cache of workspaces
// is set up once.
#include "ctx.hpp"
#include "hip_stub.hpp"

namespace {

// No host memory for the cache's own bookkeeping: contexts work without it.
void no_host_memory() {
  for (size_t good = 0;; ++good) {
    aqt_ctx* c = nullptr;
    stub::host_allocations = good;
    const aqt_status s = aqt_create(&c, 0, nullptr);   // must not throw
    stub::host_allocations = ~size_t(0);
    if (s == AQT_OK) {
      aqt_destroy(c);
      if (good > 8) break;
    } else {
      CHECK(s == AQT_ENOMEM && !c);
    }
  }
}

}  // namespace

int main() {
  no_host_memory();
  return 0;
}
