// Quad-lane chain rollout kernels (5..8 links) and their launch.  The units that
// include this differ in their scheduling options only, and in GEN, which keeps
// their kernels apart.
#pragma once

#include "kernels.hpp"
#include "rollout_grid.hpp"

namespace mtp {

template <int N, bool ONE, bool GEN>
__global__ __launch_bounds__(kRollThreads) MTP_ROLL_WAVES(ONE) void k_rollout_chain_quad(PlanDesc P) {
  if (static_cast<int>(blockIdx.x) >= P.roll_blocks) { gen_tensor_tiles(P); return; }
  const int g = xcd_contiguous_block(blockIdx.x, P.roll_blocks) * kRollThreads + threadIdx.x;
  const int b = g >> 2;
  if (b < P.B) rollout_chain_quad<N>(P, b, g & 3);
}

}  // namespace mtp
