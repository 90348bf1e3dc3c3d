// Rule and launcher of the wide rollout forms (rollout_wide.hpp), and the line
// forms with contact.  The other forms are units of their own, as they come out
// faster under other scheduling options (build.py).
#include "rollout_wide_kernel.hpp"

namespace mtp {

int wide_blocks(const PlanDesc& P, int lanes) {
  const int cands = wide_cands(lanes, P.R);
  return (P.B + cands - 1) / cands;
}

// Lanes per candidate: the most whose launch still gives every workgroup (four
// waves) a compute unit of its own, next to kMinGenBlocks units that draw the
// next tensor paths where the plan draws ahead.  A launch of one wave per SIMD
// takes one wave's time whatever its size, which more lanes shorten; a second
// wave on a SIMD costs more than the lanes save, because the solver's row
// passes issue for every lane (64 steps, us per launch: 24 links, 4000
// candidates 222 -> 150 on four lanes -> 115 on eight; 14500 candidates 222
// against 264 on eight lanes, 1812 waves).  Plain chains of two and three
// links stay narrow: moving three rows across lanes costs what it saves
// (3 links, 561 candidates: 30.6 us narrow, 33.0 on four lanes).  Randomised
// models always run side by side, on the narrow form's lanes if need be.
int wide_lanes(const PlanDesc& P) {
  if (P.dyn == kPointMass || is_quad_chain(P.dyn, P.n_links)) return 0;
  const bool pair = is_pair_chain(P.dyn, P.n_links);
  if (!pair && P.dyn == kChain && P.n_links < 4) return 0;
  const int narrow = pair ? 2 : 1;
  const int most = pair ? (P.n_links % 8 == 0 ? 8 : (P.n_links % 4 == 0 ? 4 : 2)) : 4;
  const int units = P.gen_grid - (P.U2 != nullptr ? kMinGenBlocks : 0);
  int best = P.R > 1 ? narrow : 0;
  for (int lanes = P.R > 1 ? narrow : 2 * narrow; lanes <= most; lanes *= 2)
    if (wide_blocks(P, lanes) <= units) best = lanes;
  return best;
}

hipError_t launch_rollout_wide(const PlanDesc& P, int lanes, dim3 grid, size_t lds, hipStream_t st, bool one) {
  const bool pair = is_pair_chain(P.dyn, P.n_links);
  if (P.dyn == kChain)
    return pair ? launch_wide_half(P, lanes, grid, lds, st, one) : launch_wide_rest(P, lanes, grid, lds, st, one);
  if (pair) return launch_wide_rest(P, lanes, grid, lds, st, one);
  switch (P.n_links) {
#define X(N) case N: return launch_line<N, true>(P, lanes, grid, lds, st, one);
    MTP_CONTACT_LINKS(X)
#undef X
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mtp
