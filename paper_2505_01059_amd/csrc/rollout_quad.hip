// Quad-lane rollouts, and the choice between them and those of a launch that is as
// long as its generator (rollout_quad_gen.hip).
#include "rollout_quad.hpp"

namespace mtp {

// The generator's loops are a third longer under this unit's option than under
// rollout_quad_gen.hip's, the rollout up to 2 % shorter (7 links, us per replan of
// four iterations here and there: 9216 candidates x 128 steps 505 and 510; 14000 x
// 128 799 and 578; 13000 x 64 340 and 307; 16 steps 11000 149 and 141, 10000 140
// and 140).  Only loops of a fixed length differ (linear paths 583 and 592).
static bool gen_bound(const PlanDesc& P, int blocks) {
  const int gens = blocks - P.roll_blocks;
  return gens > 0 && (P.interp == kAkima || (P.interp == kBspline && P.p == 3)) && gen_us(P, gens) > narrow_wave_us(P);
}

hipError_t launch_rollout_quad(const PlanDesc& P, dim3 grid, size_t lds, hipStream_t st, bool one) {
  if (one && gen_bound(P, static_cast<int>(grid.x))) return launch_rollout_quad_gen(P, grid, lds, st);
  switch (P.n_links) {
#define X(N)                                                                              \
  case N:                                                                                 \
    if constexpr (quad_chain_links<N>()) {                                                \
      if (one) k_rollout_chain_quad<N, true, false><<<grid, kRollThreads, lds, st>>>(P);  \
      else k_rollout_chain_quad<N, false, false><<<grid, kRollThreads, lds, st>>>(P);     \
      return hipGetLastError();                                                           \
    }                                                                                     \
    break;
    MTP_CHAIN_LINKS(X)
#undef X
    default: break;
  }
  return hipErrorInvalidValue;
}

}  // namespace mtp
