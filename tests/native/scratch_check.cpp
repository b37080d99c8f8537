// The workspace cache (csrc/scratch.hip, ScratchBuf) behind a stubbed device allocator: every
// block's true size is known here, so a block handed out below the size asked for is an error.
#include <memory>
#include <mutex>
#include <random>
#include <set>
#include <thread>
#include <vector>

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

// Blocks stay within the cache's bound, oldest out first, and go back to the device when an
// allocation needs them, when the program asks, and with the last context.
void idle_blocks() {
  aqt_ctx* c[2];
  for (aqt_ctx*& k : c) CHECK(aqt_create(&k, 0, nullptr) == AQT_OK);
  const size_t held = stub::used;   // by the contexts themselves
  {
    std::vector<std::unique_ptr<ScratchBuf>> bufs;
    for (size_t k = 0; k < 20; ++k) {   // all out at once
      bufs.push_back(std::make_unique<ScratchBuf>(c[k & 1]));
      take(*bufs.back(), size_t(1) << 30);
    }
    CHECK(stub::used - held == size_t(20) << 30);
  }
  CHECK(stub::used - held == size_t(16) << 30);
  stub::limit = stub::used;
  {
    ScratchBuf big(c[0]);   // fits no idle block
    CHECK(big.reserve((size_t(16) << 30) + 1) != hipSuccess);
    take(big, size_t(15) << 30);   // only with the idle blocks given back
    CHECK(stub::used - held == size_t(15) << 30);
  }
  stub::limit = size_t(288) << 30;
  CHECK(stub::used - held == size_t(15) << 30);
  CHECK(aqt_release_workspaces(1) == AQT_EINVAL && aqt_release_workspaces(-1) == AQT_EINVAL);
  CHECK(stub::used - held == size_t(15) << 30);
  CHECK(aqt_release_workspaces(0) == AQT_OK);
  CHECK(stub::used == held);
  {
    ScratchBuf b(c[0]);
    take(b, 1 << 20);
  }
  aqt_destroy(c[0]);
  CHECK(stub::used > (1 << 20));   // the other context keeps it
  aqt_destroy(c[1]);
  CHECK(stub::used == 0);
}

// Several threads with a context each; their blocks never overlap.
void threads() {
  std::mutex m;
  std::set<char*> out;
  std::vector<std::thread> pool;
  for (int t = 0; t < 4; ++t)
    pool.emplace_back([&, t] {
      aqt_ctx ctx;
      aqt::scratch_context(0, 1);
      std::mt19937 rng(t);
      for (int k = 0; k < 2000; ++k) {
        ScratchBuf a(&ctx), b(&ctx);
        CHECK(a.reserve(1 + rng() % (1 << 20)) == hipSuccess && b.reserve(1 + rng() % (1 << 20)) == hipSuccess);
        if (k & 1) a.swap(b);
        {
          std::lock_guard<std::mutex> lock(m);
          CHECK(out.insert(a.as<char>()).second && out.insert(b.as<char>()).second);
        }
        std::this_thread::yield();
        {
          std::lock_guard<std::mutex> lock(m);
          out.erase(a.as<char>());
          out.erase(b.as<char>());
        }
      }
      aqt::scratch_context(0, -1);
    });
  for (std::thread& t : pool) t.join();
  CHECK(stub::used == 0);
}

}  // namespace

int main() {
  mixed_sizes();
  idle_blocks();
  threads();
  std::puts("ok");
  return 0;
}
