// Packed step operands when their packing fails half way.
#include "host_check.hpp"

namespace {

aqt_status run(aqt_ctx* c, int precision) {
  aqt_run_params p{};
  p.precision = precision;
  p.n_traj = 64;
  aqt_outputs o{};
  return aqt_run(c, &p, &o);
}

// Whichever allocation of a change of precision fails, operands of the earlier precision that
// were overwritten or given up are not taken for resident afterwards.
void failed_packing() {
  const int precisions[] = {AQT_FP64, AQT_FP32, AQT_BF16};
  for (int from : precisions)
    for (int to : precisions) {
      if (from == to) continue;
      for (size_t room = 0; room < (size_t(4) << 20); room += 4096) {
        aqt_ctx* c = context_with_tables(128, 7, 20);
        CHECK(run(c, from) == AQT_OK && c->packed_for == from);
        stub::limit = stub::used + room;
        const aqt_status s = run(c, to);
        stub::limit = size_t(288) << 30;
        if (s == AQT_OK) {
          aqt_destroy(c);
          break;
        }
        CHECK(s == AQT_ENOMEM);
        stub::calls.clear();
        CHECK(run(c, from) == AQT_OK);
        CHECK(stub::count("k_pack") > 0);   // packed again
        aqt_destroy(c);
      }
    }
}

}  // namespace

int main() {
  failed_packing();
  return 0;
}
