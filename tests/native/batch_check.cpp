// Tile widths that a batch chooses up to 32 levels.
#include "host_check.hpp"

namespace {

// The widths of a batch of n instances of K trajectories each; *timed counts trajectory
// launches during its creation.
std::vector<int32_t> widths(int levels, int precision, int n, int64_t K, int flags, int tile = 0, size_t* timed = nullptr) {
  std::vector<aqt_ctx*> c;
  for (int i = 0; i < n; ++i) c.push_back(context_with_tables(levels, 4, 3));
  std::vector<aqt_run_params> p(n);
  std::vector<aqt_outputs> o(n);
  for (auto& q : p) {
    q = aqt_run_params{};
    q.precision = precision;
    q.n_traj = K;
    q.tile = tile;
  }
  stub::calls.clear();
  aqt_batch* b = nullptr;
  CHECK(aqt_batch_create(&b, c.data(), n, p.data(), o.data(), flags) == AQT_OK);
  if (timed) *timed = stub::count("k_batch");
  std::vector<int32_t> t(n);
  CHECK(aqt_batch_tiles(b, t.data()) == AQT_OK);
  aqt_batch_destroy(b);
  for (aqt_ctx* k : c) aqt_destroy(k);
  for (int32_t v : t) CHECK(v == t[0]);
  return t;
}

// Columns of 8 trajectories that a launch of the stub's 256 CUs takes: up to 8 a CU in tiles of 4,
// up to 256 a CU in tiles of 8, else of 16.
void chosen_widths() {
  for (int levels : {4, 16, 32})
    for (int precision : {AQT_FP64, AQT_FP32, AQT_BF16})
      for (int flags : {0, int(AQT_BATCH_AUTOTUNE)}) {
        size_t timed = 0;
        CHECK(widths(levels, precision, 2, 8 * 1024, flags, 0, &timed)[0] == 4 && timed == 0);
        CHECK(widths(levels, precision, 2, 8 * 1024 + 1, flags, 0, &timed)[0] == 8 && timed == 0);
        CHECK(widths(levels, precision, 2, 8 * 32768, flags, 0, &timed)[0] == 8 && timed == 0);
        CHECK(widths(levels, precision, 2, 8 * 32768 + 1, flags, 0, &timed)[0] == 16 && timed == 0);
        for (int tile : {4, 8, 16, 32, 64}) CHECK(widths(levels, precision, 2, 100, flags, tile)[0] == tile);
      }
}

// Sums that do not fit with the chosen width take the next wider one; an explicit width does not.
void widths_that_fit() {
  const int64_t K = 8 * 32768, M = 400;
  for (int tile : {8, 16, 32, 64}) {
    aqt_ctx* c = context_with_tables(16, 4, M);
    aqt_run_params p{};
    p.precision = AQT_FP32;
    p.n_traj = 8;
    aqt_outputs o{};
    CHECK(aqt_run(c, &p, &o) == AQT_OK);   // operands resident
    c->partial.release();
    p.n_traj = K;
    aqt_batch* b = nullptr;
    const size_t room = K / tile * M * 16, items = 1 << 20;
    stub::limit = stub::used + room + items;
    CHECK(aqt_batch_create(&b, &c, 1, &p, &o, 0) == AQT_OK);
    int32_t t = 0;
    CHECK(aqt_batch_tiles(b, &t) == AQT_OK && t == tile);
    aqt_batch_destroy(b);
    c->partial.release();
    if (tile > 8) {
      p.tile = 8;
      CHECK(aqt_batch_create(&b, &c, 1, &p, &o, 0) == AQT_ENOMEM);
      aqt_batch_destroy(b);
    }
    stub::limit = size_t(288) << 30;
    aqt_destroy(c);
  }
}

// The width that a batch reports is accepted as an explicit one, by batches and runs; 4 only up
// to 32 levels, where it means that many.
void width_of_four() {
  for (int levels : {4, 32, 33, 256}) {
    aqt_ctx* c = context_with_tables(levels, 4, 3);
    aqt_run_params p{};
    p.precision = AQT_FP64;
    p.n_traj = 101;
    p.tile = 4;
    aqt_outputs o{};
    const aqt_status want = levels <= 32 ? AQT_OK : AQT_EINVAL;
    stub::calls.clear();
    CHECK(aqt_run(c, &p, &o) == want);
    for (const stub::Call& k : stub::calls)
      if (k.name.find("k_trajectories") != std::string::npos) CHECK(k.grid.x == 26);
    CHECK(stub::count("k_trajectories") == (levels <= 32 ? 1u : 0u));
    aqt_batch* b = nullptr;
    CHECK(aqt_batch_create(&b, &c, 1, &p, &o, 0) == want);
    aqt_batch_destroy(b);
    for (int tile : {1, 2, 3, 5, 6, 12, -4}) {
      p.tile = tile;
      CHECK(aqt_run(c, &p, &o) == AQT_EINVAL);
      CHECK(aqt_batch_create(&b, &c, 1, &p, &o, 0) == AQT_EINVAL);
      aqt_batch_destroy(b);
    }
    aqt_destroy(c);
  }
}

// A batch's per-tile sums are its own: a larger run of a member (also of one that is in the batch
// twice) frees nothing that the batch's launches use.
void sums_of_its_own() {
  aqt_ctx* c[3] = {context_with_tables(16, 4, 50), context_with_tables(64, 4, 50), nullptr};
  c[2] = c[0];
  aqt_run_params p[3]{};
  aqt_outputs o[3]{};
  for (int k = 0; k < 3; ++k) {
    p[k].precision = AQT_FP64;
    p[k].n_traj = 100 + 1000 * k;
  }
  aqt_batch* b = nullptr;
  CHECK(aqt_batch_create(&b, c, 3, p, o, 0) == AQT_OK);
  const auto live = stub::live;
  for (int k = 0; k < 2; ++k)
    for (int64_t K : {1000, 100000}) {
      p[k].n_traj = K;
      CHECK(aqt_run(c[k], &p[k], &o[k]) == AQT_OK);
    }
  size_t gone = 0;
  for (const auto& l : live) gone += !stub::live.count(l.first);
  CHECK(gone == 0);
  CHECK(aqt_batch_launch(b) == AQT_OK);
  aqt_batch_destroy(b);
  for (int k = 0; k < 2; ++k) aqt_destroy(c[k]);
}

// Above 32 levels autotuning times every width (the stub's clock stands still: the first).
void timed_widths() {
  size_t timed = 0;
  CHECK(widths(64, AQT_FP32, 2, 1000, AQT_BATCH_AUTOTUNE, 0, &timed)[0] == 8 && timed > 2);
  CHECK(widths(64, AQT_FP32, 2, 1000, 0, 0, &timed)[0] == 32 && timed == 0);
}

}  // namespace

int main() {
  chosen_widths();
  widths_that_fit();
  width_of_four();
  sums_of_its_own();
  timed_widths();
  return 0;
}
