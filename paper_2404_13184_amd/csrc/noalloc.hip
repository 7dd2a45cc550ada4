// tanq_sample_noalloc: all-qubit sampling that allocates nothing, for callers that cannot call
// hipMalloc (tight serving loops, harnesses that forbid it).  The CDF is formed in the handle's scratch and
// up to 2^17 outcomes pass through its pinned result buffer, so calls on different handles are
// independent of each other.
#include "abi_util.hpp"

extern "C" tanq_status tanq_sample_noalloc(tanq_dm d, uint64_t shots, uint64_t seed, const double* p01,
                                           const double* p10, uint64_t* host_out) {
  return tanq::guarded([&] {
    int n = 0, device = 0;
    bool own = false;
    tanq::sample_check(d, shots, seed, p01, p10, host_out, &n, &device, &own);
    if (!own)
      tanq::fail(TANQ_E_ARG, "tanq_sample_noalloc draws at most 2^17 shots per call; asked for " + std::to_string(shots));
    if (shots == 0) return;
    tanq::sample_run(d, shots, seed, p01, p10, nullptr, host_out);
  });
}
