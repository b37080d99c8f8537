// Tile widths of a run: what its per-tile sums may take.
#include "host_check.hpp"

namespace {

constexpr size_t kCard = size_t(288) << 30;

// Workgroups of the run's trajectory launches.
struct Launch {
  aqt_status status;
  unsigned groups = 0;
};
Launch run(aqt_ctx* c, int precision, int64_t K, int tile = 0) {
  aqt_run_params p{};
  p.precision = precision;
  p.n_traj = K;
  p.tile = tile;
  aqt_outputs o{};
  stub::calls.clear();
  Launch r{aqt_run(c, &p, &o)};
  for (const stub::Call& k : stub::calls)
    if (k.name.find("k_trajectories") != std::string::npos) r.groups += k.grid.x;
  return r;
}

// A run whose sums do not fit with the fastest width takes the narrowest wider tile with which
// they do: 32 trajectories, or 64, up to 32 levels.
void falls_back_to_wide_tiles() {
  const int64_t K = 4000000, M = 400;
  for (int levels : {4, 16, 32})
    for (int precision : {AQT_FP64, AQT_FP32, AQT_BF16}) {
      aqt_ctx* c = context_with_tables(levels, 5, M);
      CHECK(run(c, precision, 8).status == AQT_OK);   // operands resident
      const Launch all = run(c, precision, K);
      CHECK(all.status == AQT_OK && all.groups == K / 16);
      for (int tile : {32, 64}) {
        c->partial.release();
        const size_t room = K / tile * M * 16;
        stub::limit = stub::used + room;
        const Launch few = run(c, precision, K);
        CHECK(few.status == AQT_OK && few.groups == K / tile);
        c->partial.release();
        CHECK(run(c, precision, K, 16).status == AQT_ENOMEM);   // an explicit width is kept
        stub::limit = kCard;
      }
      c->partial.release();
      stub::limit = stub::used + K / 64 * M * 16 - 1;
      CHECK(run(c, precision, K).status == AQT_ENOMEM);
      stub::limit = kCard;
      aqt_destroy(c);
    }
}

// Sums beyond 4 GiB take tiles of 32 although there is room.
void large_sums_take_wide_tiles() {
  const int64_t M = 50, K = (int64_t(4) << 30) / M / 16 * 16;
  aqt_ctx* c = context_with_tables(16, 4, M);
  CHECK(run(c, AQT_FP32, K).groups == K / 16);
  CHECK(run(c, AQT_FP32, K + 16).groups == (K + 16 + 31) / 32);
  aqt_destroy(c);
}

}  // namespace

int main() {
  falls_back_to_wide_tiles();
  large_sums_take_wide_tiles();
  return 0;
}
