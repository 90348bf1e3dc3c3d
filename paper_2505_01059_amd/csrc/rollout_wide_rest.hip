// Wide half forms with contact, and line forms without.
#include "rollout_wide_kernel.hpp"

namespace mtp {

hipError_t launch_wide_rest(const PlanDesc& P, int lanes, dim3 grid, size_t lds, hipStream_t st, bool one) {
  if (P.dyn == kChain) {
    switch (P.n_links) {
#define X(N) case N: return launch_line<N, false>(P, lanes, grid, lds, st, one);
      MTP_CHAIN_LINKS(X)
#undef X
      default: return hipErrorInvalidValue;
    }
  }
  switch (P.n_links) {
#define X(N) case N: return launch_half<N, true>(P, lanes, grid, lds, st, one);
    MTP_CONTACT_LINKS(X)
#undef X
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mtp
