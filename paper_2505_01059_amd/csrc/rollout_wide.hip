// Kernels and launcher of the wide rollout forms (rollout_wide.hpp).
#include "kernels.hpp"
#include "rollout_grid.hpp"
#include "rollout_wide.hpp"

namespace mtp {

// A wide form: lanes per candidate and randomised model, the lane of a group
// whose cost is written, and the rollout itself.
template <int N, int S, bool CONTACT, bool EQ>
struct HalfForm {
  static constexpr int kLanes = 2 * S, kWriter = S - 1;
  static __device__ __forceinline__ float cost(const PlanDesc& P, int b, int pos, int rep, bool live) {
    return rollout_half<N, S, CONTACT, EQ>(P, b, pos, rep, live);
  }
};
template <int N, int L, bool CONTACT>
struct LineForm {
  static constexpr int kLanes = L, kWriter = L - 1;
  static __device__ __forceinline__ float cost(const PlanDesc& P, int b, int pos, int rep, bool live) {
    return rollout_line<N, L, CONTACT>(P, b, pos, rep, live);
  }
};

// Candidates per workgroup: the groups of a workgroup hold every candidate
// under as many randomised models at a time as fit.
__host__ __device__ constexpr int wide_models(int lanes, int R) { return R < kRollThreads / lanes ? R : kRollThreads / lanes; }
__host__ __device__ constexpr int wide_cands(int lanes, int R) { return kRollThreads / lanes / wide_models(lanes, R); }

// The models of a candidate run side by side in one workgroup (the narrow
// forms run them one after another); its costs meet in LDS and are summed in
// model order, as the narrow forms do.
template <class Form, bool ONE>
__global__ __launch_bounds__(kRollThreads) MTP_ROLL_WAVES(ONE) void k_rollout_wide(PlanDesc P) {
  if (static_cast<int>(blockIdx.x) >= P.roll_blocks) { gen_tensor_tiles(P); return; }
  constexpr int kLanes = Form::kLanes;
  __shared__ float sums[kRollThreads / kLanes];
  const int R = P.R;
  const int models = wide_models(kLanes, R), cands = wide_cands(kLanes, R);
  const int group = static_cast<int>(threadIdx.x) / kLanes, pos = static_cast<int>(threadIdx.x) % kLanes;
  const int m = group / cands, cl = group - m * cands;
  const int bb = xcd_contiguous_block(blockIdx.x, P.roll_blocks) * cands + cl;
  const bool in = bb < P.B && m < models;
  const int b = bb < P.B ? bb : P.B - 1;   // idle groups shadow the last candidate and store nothing
  if (R == 1) {
    const float cost = Form::cost(P, b, pos, 0, in);
    if (in && pos == Form::kWriter) P.cost[b] = finite_or_inf(cost);
    return;
  }
  float total = 0.0f;
  for (int r0 = 0; r0 < R; r0 += models) {
    const int rep = min(r0 + m, R - 1);
    const bool live = in && r0 + m < R;
    const float cost = Form::cost(P, b, pos, rep, live);
    if (pos == Form::kWriter) sums[group] = cost;
    __syncthreads();
    if (m == 0 && pos == Form::kWriter)
      for (int i = 0; i < models && r0 + i < R; ++i) total += sums[i * cands + cl];
    __syncthreads();
  }
  if (in && m == 0 && pos == Form::kWriter) P.cost[b] = finite_or_inf(total / static_cast<float>(R));
}

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
// candidates 222 -> 150 on four lanes -> 126 on eight; 14500 candidates 222
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

template <class Form>
static hipError_t launch_form(const PlanDesc& P, dim3 grid, size_t lds, hipStream_t st) {
  k_rollout_wide<Form, true><<<grid, kRollThreads, lds, st>>>(P);
  return hipGetLastError();
}

template <class Form>
static hipError_t launch_narrow(const PlanDesc& P, dim3 grid, size_t lds, hipStream_t st, bool one) {
  if (one) return launch_form<Form>(P, grid, lds, st);
  k_rollout_wide<Form, false><<<grid, kRollThreads, lds, st>>>(P);
  return hipGetLastError();
}

template <int N, bool CONTACT>
static hipError_t launch_n(const PlanDesc& P, int lanes, dim3 grid, size_t lds, hipStream_t st, bool one) {
  if constexpr (pair_chain_links<N>()) {
    if constexpr (CONTACT)
      if (lanes == 2)
        return P.eq_len ? launch_narrow<HalfForm<N, 1, CONTACT, true>>(P, grid, lds, st, one)
                        : launch_narrow<HalfForm<N, 1, CONTACT, false>>(P, grid, lds, st, one);
    if constexpr (N % 4 == 0)
      if (lanes == 4)
        return P.eq_len ? launch_form<HalfForm<N, 2, CONTACT, true>>(P, grid, lds, st)
                        : launch_form<HalfForm<N, 2, CONTACT, false>>(P, grid, lds, st);
    if constexpr (N % 8 == 0)
      if (lanes == 8)
        return P.eq_len ? launch_form<HalfForm<N, 4, CONTACT, true>>(P, grid, lds, st)
                        : launch_form<HalfForm<N, 4, CONTACT, false>>(P, grid, lds, st);
  } else if constexpr (CONTACT || (N >= 4 && !quad_chain_links<N>())) {
    if constexpr (CONTACT)
      if (lanes == 1) return launch_narrow<LineForm<N, 1, CONTACT>>(P, grid, lds, st, one);
    if (lanes == 2) return launch_form<LineForm<N, 2, CONTACT>>(P, grid, lds, st);
    if (lanes == 4) return launch_form<LineForm<N, 4, CONTACT>>(P, grid, lds, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_rollout_wide(const PlanDesc& P, int lanes, dim3 grid, size_t lds, hipStream_t st, bool one) {
  if (P.dyn == kChain) {
    switch (P.n_links) {
#define X(N) case N: return launch_n<N, false>(P, lanes, grid, lds, st, one);
      MTP_CHAIN_LINKS(X)
#undef X
      default: return hipErrorInvalidValue;
    }
  }
  switch (P.n_links) {
#define X(N) case N: return launch_n<N, true>(P, lanes, grid, lds, st, one);
    MTP_CONTACT_LINKS(X)
#undef X
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mtp
