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
  stub::on_download = [&](void* dst, const void*, size_t n) {
    if (n == sizeof(int)) *static_cast<int*>(dst) = 1;   // the ground state of H(0) is not degenerate
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

}  // namespace

int main() {
  failed_heads(0);
  failed_heads(1);

  return 0;
}
