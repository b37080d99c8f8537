// Chains of the iterative eigensolver when their joint start fails or memory is short.  On the
// stubbed runtime every residual is zero, so each solve ends after one iteration.
#include "host_check.hpp"

namespace {

aqt_ctx* iterative_context() {
  aqt_ctx* c = nullptr;
  CHECK(aqt_create(&c, 0, nullptr) == AQT_OK);
  const int nq = 7;
  const std::vector<double> h(nq, 0.5), J(nq * nq, 0.1), A{1.0, 0.0}, B{0.0, 1.0};
  CHECK(aqt_set_hamiltonian(c, nq, h.data(), J.data()) == AQT_OK);
  CHECK(aqt_set_schedule(c, 10.0, 2, A.data(), B.data()) == AQT_OK);
  CHECK(aqt_set_bath(c, 1e-4, 50.0, 1.5) == AQT_OK);
  return c;
}

constexpr int kPoints = 6000;   // more than one chunk (65535 / 14 grid points)
constexpr size_t kSlots = 64;

// The joint solve of the chain heads of chunk `chunk` (0 or 1) fails once: the heads are then
// solved one after another, the first from a random block, and nothing is left of the failure.
void failed_heads(int chunk) {
  aqt_ctx* c = iterative_context();
  size_t random = 0, after = 0, failures = 0;
  bool armed = false;
  // random starts: every head of the first chunk, all but the first of the second
  const size_t at = chunk ? 2 * kSlots - 1 : kSlots;
  stub::on_call = [&](const stub::Call& k) {
    if (k.name.find("k_random_block") == std::string::npos) return;
    ++random;
    if (failures) ++after;
    armed = armed || random == at;
  };
  stub::on_download = [&](void* dst, const void* src, size_t n) {
    if (src == c->gs.p) *static_cast<int*>(dst) = 1;   // the ground state of H(0) is not degenerate
    if (armed && !failures && n == kSlots * sizeof(int)) {   // per-slot status of the small eigenproblems
      static_cast<int*>(dst)[0] = 1;
      ++failures;
    }
  };
  const aqt_status s = aqt_precompute_ex(c, kPoints, 16, 1e-8, AQT_EIG_ITERATIVE);
  stub::on_call = nullptr;
  stub::on_download = nullptr;
  if (s != AQT_OK) std::printf("%d %s %zu %zu\n", s, aqt_last_error(c), random, failures);
  CHECK(s == AQT_OK && failures == 1);
  // the first head again from a random block, and for the first chunk the next one's others
  CHECK(after == (chunk ? 1 : 1 + kSlots - 1));
  CHECK(std::string(aqt_last_error(c)).empty());
  aqt_destroy(c);
}

// Chains solved together, by the random blocks they start from, within the memory there is.
size_t chains_within(size_t room, aqt_status* status, int points = 200) {
  aqt_ctx* c = iterative_context();
  size_t random = 0;
  stub::on_call = [&](const stub::Call& k) { random += k.name.find("k_random_block") != std::string::npos; };
  stub::on_download = [&](void* dst, const void* src, size_t) {
    if (src == c->gs.p) *static_cast<int*>(dst) = 1;
  };
  stub::peak = stub::used;
  const size_t before = stub::used;
  stub::limit = room ? before + room : size_t(288) << 30;
  *status = aqt_precompute_ex(c, points, 16, 1e-8, AQT_EIG_ITERATIVE);
  stub::limit = size_t(288) << 30;
  stub::on_call = nullptr;
  stub::on_download = nullptr;
  aqt_destroy(c);
  return random;
}

// Block slots that do not fit are halved, down to one, before the call gives up.
void fewer_slots_in_less_memory() {
  aqt_status s;
  size_t last = chains_within(0, &s), seen = 1;
  CHECK(s == AQT_OK && last == kSlots);
  for (size_t room = stub::peak - 1;; room -= 1 << 18) {
    const size_t now = chains_within(room, &s);
    if (s != AQT_OK) break;
    CHECK(now == last || now == last / 2);
    seen += now != last;
    last = now;
  }
  CHECK(s == AQT_ENOMEM && last == 1 && seen == 7);
}

// A short grid takes the slots of its own chains (of two points and more) alone.
void slots_of_a_short_grid() {
  aqt_status s;
  size_t peak[2];
  for (int k = 0; k < 2; ++k) {
    const size_t before = stub::used;
    CHECK(chains_within(0, &s, k ? 128 : 8) == (k ? 64 : 4) && s == AQT_OK);
    peak[k] = stub::peak - before;
  }
  CHECK(8 * peak[0] < peak[1]);
}

}  // namespace

int main() {
  failed_heads(0);
  failed_heads(1);
  fewer_slots_in_less_memory();
  slots_of_a_short_grid();
  return 0;
}
