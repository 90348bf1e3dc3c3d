// Time-sliced pair-lane rollout kernels (long chains whose pair-lane waves
// outnumber the SIMDs) and their launcher.  A unit of its own so that it can be
// compiled with its own scheduling options.
#include <algorithm>

#include "kernels.hpp"
#include "rollout_grid.hpp"

namespace mtp {

// Every wave of the grid is a worker.
constexpr uint64_t kSegWaitTicks = 1000000000ull;   // 10 s of the 100 MHz wall clock

// EQ: every link has the same length (P.eq_len), held once instead of per link.
template <int N, bool CONTACT, bool EQ>
__global__ __launch_bounds__(kRollThreads) MTP_ROLL_WAVES(true) void k_rollout_pair_seg(PlanDesc P) {
  rollout_pair_segmented<N, CONTACT, EQ>(P, P.seg_ctl, P.seg_done, P.seg_state, P.seg_S, P.seg_len, kSegWaitTicks);
  if (threadIdx.x == 0 && __hip_atomic_load(&P.seg_ctl->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u)
    atomicOr(&P.ctrl[2], 4u);
}

// New launch of the time-sliced rollout: next epoch, unit counter and error cleared.
__global__ __launch_bounds__(64) void k_seg_init(SegCtl* ctl) {
  if (threadIdx.x == 0) {
    ctl->head = 0u;
    ctl->error = 0u;
    ctl->epoch = ctl->epoch + 1u;
  }
}

hipError_t launch_rollout_seg(const PlanDesc& P, hipStream_t st) {
  k_seg_init<<<1, 64, 0, st>>>(P.seg_ctl);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const size_t lds = seg_lds_bytes(P);
  if (P.dyn == kChain) {
    switch (P.n_links) {
#define X(N)                                                                                         \
  case N:                                                                                            \
    if constexpr (pair_chain_links<N>()) {                                                           \
      if (P.eq_len) k_rollout_pair_seg<N, false, true><<<P.seg_grid, kRollThreads, lds, st>>>(P);      \
      else k_rollout_pair_seg<N, false, false><<<P.seg_grid, kRollThreads, lds, st>>>(P);              \
      return hipGetLastError();                                                                      \
    }                                                                                                \
    break;
      MTP_CHAIN_LINKS(X)
#undef X
      default: break;
    }
    return hipErrorInvalidValue;
  }
  switch (P.n_links) {
#define X(N)                                                                                         \
  case N:                                                                                            \
    if constexpr (pair_chain_links<N>()) {                                                           \
      if (P.eq_len) k_rollout_pair_seg<N, true, true><<<P.seg_grid, kRollThreads, lds, st>>>(P);       \
      else k_rollout_pair_seg<N, true, false><<<P.seg_grid, kRollThreads, lds, st>>>(P);               \
      return hipGetLastError();                                                                      \
    }                                                                                                \
    break;
    MTP_CONTACT_LINKS(X)
#undef X
    default: break;
  }
  return hipErrorInvalidValue;
}

// Workers: one wave per SIMD, and no more than there are wave groups.  A worker
// beyond the groups takes a segment whose predecessor has only just begun and
// waits a whole segment's time for it, its polling taking the caches from the
// others (12 links, 40000 candidates x 64 steps, 1250 groups: on the 2048 waves
// that fit by registers 1825 us per launch, on 1024 546 us, and 220 us since the
// state goes past the L2 caches).
hipError_t seg_configure(PlanDesc* P) {
  if (P->seg_ctl == nullptr) return hipSuccess;
  int dev = 0, grid = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&grid, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  constexpr int kWaves = kRollThreads / 64;
  const int groups = (P->B + 31) / 32;
  grid = std::max(1, std::min(grid, groups / kWaves));
  const double step_us = (P->dyn == kChainContact ? 0.22 : 0.14) * P->n_links;
  P->seg_S = segment_count(groups, grid * kWaves, P->T, step_us);
  P->seg_len = (P->T + P->seg_S - 1) / P->seg_S;
  P->seg_S = (P->T + P->seg_len - 1) / P->seg_len;   // no empty trailing segment
  P->seg_grid = grid;
  return hipSuccess;
}

}  // namespace mtp
