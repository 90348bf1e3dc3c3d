// One-lane rollout kernels of the short chains without contact and their launcher.
// A unit of its own so that it can be compiled with its own scheduling options.
#include "kernels.hpp"
#include "rollout_grid.hpp"

namespace mtp {

// One build: under this unit's option the two come out alike.
hipError_t launch_rollout_line(const PlanDesc& P, dim3 grid, size_t lds, hipStream_t st) {
  switch (P.n_links) {
#define X(N)                                                                     \
  case N:                                                                        \
    if constexpr (!pair_chain_links<N>() && !quad_chain_links<N>()) {            \
      k_rollout_chain<N, false, true, true><<<grid, kRollThreads, lds, st>>>(P); \
      return hipGetLastError();                                                  \
    }                                                                            \
    break;
    MTP_CHAIN_LINKS(X)
#undef X
    default: break;
  }
  return hipErrorInvalidValue;
}

}  // namespace mtp
