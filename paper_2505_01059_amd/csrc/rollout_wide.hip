// Rule and launcher of the wide rollout forms (rollout_wide.hpp), and the line
// forms with contact.  The other forms are units of their own, as they come out
// faster under other scheduling options (build.py).
#include <algorithm>

#include "rollout_wide_kernel.hpp"

namespace mtp {

int wide_blocks(const PlanDesc& P, int lanes) {
  const int cands = wide_cands(lanes, P.R);
  return (P.B + cands - 1) / cands;
}

namespace {

// Time of a wave on `lanes` lanes per candidate, of the narrow form's.
double wide_share(const PlanDesc& P, int lanes) {
  if (is_pair_chain(P.dyn, P.n_links)) return lanes <= 2 ? 1.0 : (lanes == 4 ? 0.69 : 0.52);
  return lanes <= 1 ? 1.0 : (lanes == 2 ? 0.78 : (P.dyn == kChainContact ? 0.53 : 0.73));
}

// A launch of `blocks` rollout workgroups, one per compute unit, each `wave_us`
// long, with the generator if `gen`: on the units that the last round leaves, or
// after it where these are too few.  `shared`: workgroups past the first round
// share the units with others (the one-lane forms' registers admit it), so the
// last round takes what there is of it.
double launch_us(const PlanDesc& P, int blocks, double wave_us, bool gen, bool shared = false) {
  const int rounds = blocks / P.gen_grid, rest = blocks % P.gen_grid;
  const double before = wave_us * rounds;
  const double last = rest == 0 ? 0.0 : (shared && rounds > 0 ? wave_us * rest / P.gen_grid : wave_us);
  if (!gen) return before + last;
  const int left = P.gen_grid - rest;
  return before + (left >= kMinGenBlocks ? std::max(last, gen_us(P, left)) : last + gen_us(P, kMinGenBlocks));
}

}  // namespace

double narrow_wave_us(const PlanDesc& P) {
  const bool contact = P.dyn == kChainContact;
  if (is_quad_chain(P.dyn, P.n_links)) return 0.85 * P.T;
  if (is_pair_chain(P.dyn, P.n_links)) return (contact ? 0.18 : 0.15) * P.n_links * P.T;
  return (contact ? 0.46 : 0.3) * P.n_links * P.T;
}

// Drawing 256 candidates of a joint: the graph column and the indices by layers,
// the spline by steps (9 layers, us per item at 16, 64 and 200 steps: cubic 4.1,
// 9.0, 23; Akima 10.8 at 64, 26 at 200; linear 12.5 at 64).
double gen_us(const PlanDesc& P, int gens) {
  const int first = (P.G - 1) / kCandThreads, last = (P.G - 1 + P.P - 1) / kCandThreads;
  const int items = (last - first + 1) * P.n;
  const double setup = 0.4 + 0.22 * P.L;
  const double item = P.interp == kAkima                 ? setup + 1.1 + 0.114 * P.T
                      : P.interp == kBspline && P.p == 3 ? setup + 0.103 * P.T
                                                         : setup + 0.158 * P.T;
  return ((items + gens - 1) / gens) * item;
}

// Lanes per candidate: those whose launch is estimated the shortest, beside the
// generator if `gen`; 0 is the narrow form with the randomised models in turn.
//
// A launch of one wave per SIMD takes one wave's time whatever its size, which
// more lanes shorten; past one workgroup per compute unit, a second wave on a SIMD
// costs more than the lanes save, because the solver's row passes issue for
// every lane (64 steps, us per launch: 24 links, 4000 candidates 222 -> 150 on
// four lanes -> 115 on eight; 14500 candidates 222 against 264 on eight lanes,
// 1812 waves).  The units a wide form takes are missing to the generator: 14000
// candidates of 24 links fit on four lanes beside 37 generator workgroups, which
// then take longer than the narrow rollout does (16 steps, four iterations: 340
// us narrow, 620 on four lanes; 12 links 228 and 354; 28000 candidates of 4 links
// on two lanes 261 and 341).  Randomised models side by side likewise: 18000
// candidates of 24 links in contact, two models, 665 us in turn, 1042 side by
// side; but 45800 of 7 links in contact, two models x 128 steps, 888 us an
// iteration in turn, 698 side by side, where workgroups share units.  Plain chains
// of two and three links stay narrow: moving three rows across lanes costs what it
// saves (3 links, 561 candidates: 30.6 us narrow, 33.0 on four lanes).
int wide_lanes(const PlanDesc& P, bool gen) {
  if (P.dyn == kPointMass || is_quad_chain(P.dyn, P.n_links)) return 0;
  const bool pair = is_pair_chain(P.dyn, P.n_links);
  if (!pair && P.dyn == kChain && P.n_links < 4) return 0;
  const int narrow = pair ? 2 : 1;
  const int most = pair ? (P.n_links % 8 == 0 ? 8 : (P.n_links % 4 == 0 ? 4 : 2)) : 4;
  const double wave = narrow_wave_us(P);
  constexpr double kGain = 0.95;   // of the best so far, for a wider form to be taken
  int best = 0;
  double best_us = launch_us(P, rollout_blocks(P), wave * P.R, gen);
  for (int lanes = narrow; lanes <= most; lanes *= 2) {
    const int models = wide_models(lanes, P.R), passes = (P.R + models - 1) / models;
    if (lanes == narrow && P.R == 1) continue;   // the narrow form itself
    const double us = launch_us(P, wide_blocks(P, lanes), wave * wide_share(P, lanes) * passes, gen,
                                !pair && lanes == narrow);
    if (us < kGain * best_us) {
      best = lanes;
      best_us = us;
    }
  }
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
