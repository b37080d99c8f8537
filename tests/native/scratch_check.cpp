// The workspace cache (csrc/scratch.hip, ScratchBuf) behind a stubbed device allocator: every
// block's true size is known here, so a block handed out below the size asked for is an error.
#include <random>

#include "ctx.hpp"
#include "hip_stub.hpp"

namespace {

using aqt::ScratchBuf;

void take(ScratchBuf& b, size_t n) {
  CHECK(b.reserve(n) == hipSuccess);
  CHECK(stub::live.at(b.as<char>()) >= n);
}

// Requests of the iterative eigensolver with n-state blocks, 32 levels: four blocks, the
// split-k partial products and the small matrices; `swaps` exchanges as its iterations make.
void iterative(aqt_ctx* ctx, size_t N, size_t KB, size_t slots, int swaps) {
  ScratchBuf X(ctx), Y1(ctx), Y2(ctx), W(ctx), part(ctx), S(ctx);
  const size_t blk = slots * KB * N * 8, kk = slots * KB * KB * 8;
  take(X, blk);
  take(Y1, blk);
  take(Y2, blk);
  take(W, blk);
  take(part, N / 256 * kk);
  take(S, kk);
  for (int k = 0; k < swaps; ++k) {
    X.swap(Y1);
    W.swap(Y2);
    for (ScratchBuf* b : {&X, &Y1, &Y2, &W}) CHECK(stub::live.at(b->as<char>()) >= blk);
  }
}

void mixed_sizes() {
  std::mt19937 rng(7);
  for (int parity = 0; parity < 2; ++parity) {
    aqt_ctx ctx;
    aqt::scratch_context(0, 1);
    for (const size_t nq : {12, 11, 12, 13, 12, 13, 11})
      iterative(&ctx, size_t(1) << nq, nq < 12 ? 64 : 128, 30, 16 + parity);
    for (int k = 0; k < 300; ++k) {
      const size_t nq = 10 + rng() % 4;
      iterative(&ctx, size_t(1) << nq, (rng() & 1) ? 64 : 128, 1 + rng() % 64, static_cast<int>(rng() % 20));
      ScratchBuf other(&ctx);
      take(other, 1 + rng() % (size_t(1) << 30));
    }
    aqt::scratch_context(0, -1);
    CHECK(stub::live.empty());   // the last context gives everything back
  }
}

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
  mixed_sizes();
  std::puts("ok");
  return 0;
}
