// Kernels of the wide rollout forms (rollout_wide.hpp) and their launch.  The
// units that include this differ in their scheduling options only.
#pragma once

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

// Half forms of N links: narrow (two lanes) under randomised models only.
template <int N, bool CONTACT>
static hipError_t launch_half(const PlanDesc& P, int lanes, dim3 grid, size_t lds, hipStream_t st, bool one) {
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
  }
  return hipErrorInvalidValue;
}

// Line forms of N links: one lane under randomised models only.
template <int N, bool CONTACT>
static hipError_t launch_line(const PlanDesc& P, int lanes, dim3 grid, size_t lds, hipStream_t st, bool one) {
  if constexpr (!pair_chain_links<N>() && (CONTACT || (N >= 4 && !quad_chain_links<N>()))) {
    if constexpr (CONTACT)
      if (lanes == 1) return launch_narrow<LineForm<N, 1, CONTACT>>(P, grid, lds, st, one);
    if (lanes == 2) return launch_form<LineForm<N, 2, CONTACT>>(P, grid, lds, st);
    if (lanes == 4) return launch_form<LineForm<N, 4, CONTACT>>(P, grid, lds, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace mtp
