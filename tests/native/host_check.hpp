// A context with tables on the stubbed runtime.
#pragma once

#include <vector>

#include "ctx.hpp"
#include "hip_stub.hpp"

// `levels` levels, `channels` qubits, `points` grid points; every table value is zero.
inline aqt_ctx* context_with_tables(int levels, int channels, int points, hipStream_t stream = nullptr) {
  aqt_ctx* c = nullptr;
  CHECK(aqt_create(&c, 0, stream) == AQT_OK);
  const std::vector<double> h(channels, 0.5), J(channels * channels, 0.1), A{1.0, 0.0}, B{0.0, 1.0};
  CHECK(aqt_set_hamiltonian(c, channels, h.data(), J.data()) == AQT_OK);
  CHECK(aqt_set_schedule(c, 10.0, 2, A.data(), B.data()) == AQT_OK);
  CHECK(aqt_set_bath(c, 1e-4, 50.0, 1.5) == AQT_OK);
  const size_t n = levels, M = points;
  const std::vector<double> E(M * n), O(M * n * n), ci(n), R(M * channels * n * n), z(M * channels * n);
  const std::vector<int32_t> gs(M, 1);
  CHECK(aqt_set_tables(c, points, levels, E.data(), gs.data(), O.data(), ci.data(), R.data(), z.data()) == AQT_OK);
  return c;
}
