// Quad-lane rollouts of launches that are as long as their generator, one
// workgroup per compute unit.
#include "rollout_quad.hpp"

namespace mtp {

hipError_t launch_rollout_quad_gen(const PlanDesc& P, dim3 grid, size_t lds, hipStream_t st) {
  switch (P.n_links) {
#define X(N)                                                                   \
  case N:                                                                      \
    if constexpr (quad_chain_links<N>()) {                                     \
      k_rollout_chain_quad<N, true, true><<<grid, kRollThreads, lds, st>>>(P); \
      return hipGetLastError();                                                \
    }                                                                          \
    break;
    MTP_CHAIN_LINKS(X)
#undef X
    default: break;
  }
  return hipErrorInvalidValue;
}

}  // namespace mtp
