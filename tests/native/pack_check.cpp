// Packed step operands: a packing that fails half way, and one while other streams read them.
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
      for (size_t good = 0;; ++good) {
        aqt_ctx* c = context_with_tables(128, 7, 3);
        CHECK(run(c, from) == AQT_OK && c->packed_for == from);
        stub::allocations = good;
        const aqt_status s = run(c, to);
        stub::allocations = ~size_t(0);
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

size_t first(const char* part, size_t from = 0) {
  size_t k = from;
  while (k < stub::calls.size() && stub::calls[k].name.find(part) == std::string::npos) ++k;
  return k;
}

// A batch in flight on its own stream reads the operands of a member that is then run in
// another precision: the rewriting waits for it.
void packing_under_a_batch() {
  const int precisions[] = {AQT_FP64, AQT_FP32, AQT_BF16};
  for (int from : precisions)
    for (int to : precisions) {
      if (from == to) continue;
      aqt_ctx* c[2] = {context_with_tables(16, 4, 3, reinterpret_cast<hipStream_t>(16)),
                       context_with_tables(16, 4, 3, reinterpret_cast<hipStream_t>(32))};
      aqt_run_params p[2]{};
      aqt_outputs o[2]{};
      for (auto& q : p) {
        q.precision = from;
        q.n_traj = 64;
      }
      aqt_batch* b = nullptr;
      CHECK(aqt_batch_create(&b, c, 2, p, o, 0) == AQT_OK);
      CHECK(aqt_batch_launch(b) == AQT_OK);
      stub::calls.clear();
      CHECK(run(c[1], to) == AQT_OK);
      // freeing waits for the device as well, but only some packings free a buffer
      CHECK(first("hipDeviceSynchronize") < first("k_pack") && first("k_pack") < stub::calls.size());
      aqt_batch_destroy(b);
      for (aqt_ctx* k : c) aqt_destroy(k);
    }
}

// The operands that a batch packs on its members' streams are complete before its own stream
// reads them.
void batch_waits_for_its_packings() {
  hipStream_t st[3];
  for (size_t k = 0; k < 3; ++k) st[k] = reinterpret_cast<hipStream_t>(16 * (k + 1));
  aqt_ctx* c[3];
  aqt_run_params p[3]{};
  aqt_outputs o[3]{};
  for (int k = 0; k < 3; ++k) {
    c[k] = context_with_tables(16, 4, 3, st[k]);
    p[k].precision = AQT_FP32;
    p[k].n_traj = 64;
  }
  stub::calls.clear();
  aqt_batch* b = nullptr;
  CHECK(aqt_batch_create(&b, c, 3, p, o, AQT_BATCH_AUTOTUNE) == AQT_OK);
  CHECK(aqt_batch_launch(b) == AQT_OK);
  const size_t runs = first("k_batch");
  CHECK(runs < stub::calls.size());
  for (hipStream_t s : st) {
    size_t packed = 0, waited = 0;
    for (size_t k = 0; k < runs; ++k) {
      if (stub::calls[k].stream != s) continue;
      if (stub::calls[k].name.find("k_") != std::string::npos) packed = k;
      if (stub::calls[k].name == "hipStreamSynchronize") waited = k;
    }
    CHECK(packed < waited);
  }
  aqt_batch_destroy(b);
  for (aqt_ctx* k : c) aqt_destroy(k);
}

}  // namespace

int main() {
  failed_packing();
  packing_under_a_batch();
  batch_waits_for_its_packings();
  return 0;
}
