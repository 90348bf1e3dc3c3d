// Host-callable launchers of the single-plan stage kernels (kernels.hip).
#pragma once

#include "mtp_device.hpp"

namespace mtp {

bool rollout_supported(int dyn, int n_links);
int supported_chain_links(int* out, int cap);

hipError_t launch_set_ctrl(const PlanDesc& P, uint32_t r, int shift, const float* x0_src, hipStream_t st);
hipError_t launch_shift(const PlanDesc& P, hipStream_t st);
// stage: 0 candidates, 1 rollout, 2 top-E, 3 refit (the replan index is read from P.ctrl[0])
hipError_t launch_stage(const PlanDesc& P, int stage, int k, hipStream_t st);
// A second stream that a launch sequence forks work onto and joins back from
// (fork / join events recorded on the streams; usable under graph capture).
struct SideLane {
  hipStream_t st;
  hipEvent_t fork, join;
};
// Stage of iteration k in a run of iterations [k0, k1) (next iteration's tensor
// paths drawn during the rollout when the plan has a second U buffer).  A
// time-sliced rollout fills every SIMD, so there the next tensor paths are drawn
// by a kernel of their own on `side`, beside the rollout (on `st` after it when
// side is null).
hipError_t launch_iteration_stage(const PlanDesc& P, int stage, int k, int k0, int k1, hipStream_t st,
                                  const SideLane* side = nullptr);
// The four stages of iteration k in that run, selection and refit in one launch
// where that is the faster.
hipError_t launch_iteration(const PlanDesc& P, int k, int k0, int k1, hipStream_t st, const SideLane* side = nullptr);
// Quad-lane chain rollout (rollout_quad.hip); one: the launch holds one
// workgroup per compute unit.
hipError_t launch_rollout_quad(const PlanDesc& P, dim3 grid, size_t lds, hipStream_t st, bool one);
hipError_t launch_rollout_quad_gen(const PlanDesc& P, dim3 grid, size_t lds, hipStream_t st);
// Lanes per candidate that the decision to draw ahead counts for a point mass.
constexpr int kPmOverlapLanes = 8;
// Workgroups that a drawing-ahead rollout launch adds at least.
constexpr int kMinGenBlocks = 32;
// Estimated time (us) of a wave of a chain's narrow form through the horizon, one
// wave per SIMD, and of `gens` generator workgroups.
double narrow_wave_us(const PlanDesc& P);
double gen_us(const PlanDesc& P, int gens);
// Wide rollout forms (rollout_wide.hip): the lanes per candidate a plan's
// launch takes (0: its narrow form; gen: the launch also draws ahead), the
// workgroups and the launch itself.
int wide_lanes(const PlanDesc& P, bool gen);
int wide_blocks(const PlanDesc& P, int lanes);
hipError_t launch_rollout_wide(const PlanDesc& P, int lanes, dim3 grid, size_t lds, hipStream_t st, bool one);
hipError_t launch_wide_half(const PlanDesc& P, int lanes, dim3 grid, size_t lds, hipStream_t st, bool one);
hipError_t launch_wide_rest(const PlanDesc& P, int lanes, dim3 grid, size_t lds, hipStream_t st, bool one);
// One-lane rollouts without contact (rollout_line.hip).
hipError_t launch_rollout_line(const PlanDesc& P, dim3 grid, size_t lds, hipStream_t st);
// LDS a time-sliced rollout asks for, so that no two of its workgroups share a
// compute unit: more than half of the unit's 160 KB, leaving room for a
// generator workgroup (k_gen_tensor).  From 20 links on the registers see to it.
inline size_t seg_lds_bytes(const PlanDesc& P) { return P.n_links < 20 ? 84 * 1024 : 0; }
// Time-sliced pair-lane rollout (rollout_seg.hip): epoch bump, then the
// persistent launch of P.seg_grid workgroups.
hipError_t launch_rollout_seg(const PlanDesc& P, hipStream_t st);
// A whole point-mass replan (pm_replan.hip) from start state x0_src.
hipError_t launch_pm_replan(const PlanDesc& P, uint32_t r, int shift, const float* x0_src, hipStream_t st);
// Workgroups of the (not time-sliced) rollout kernel of a plan.
int rollout_blocks(const PlanDesc& P);
// Grid and segment count of the time-sliced pair-lane rollout for the current
// device (no-op for plans that do not use it).
hipError_t seg_configure(PlanDesc* P);
// Compute units of the current device: the workgroups of a rollout launch that
// also draws the next tensor paths, and the bound below which rollout launches
// keep one workgroup per unit.
hipError_t gen_configure(PlanDesc* P);
// defined in plan.cpp
int segment_count(int groups, int resident_waves, int T, double step_us);

}  // namespace mtp
