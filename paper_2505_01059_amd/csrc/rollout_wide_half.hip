// Wide half forms of the long chains without contact.
#include "rollout_wide_kernel.hpp"

namespace mtp {

hipError_t launch_wide_half(const PlanDesc& P, int lanes, dim3 grid, size_t lds, hipStream_t st, bool one) {
  switch (P.n_links) {
#define X(N) case N: return launch_half<N, false>(P, lanes, grid, lds, st, one);
    MTP_CHAIN_LINKS(X)
#undef X
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mtp
