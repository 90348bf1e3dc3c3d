// Single-plan kernels of one MTP replan for gfx950 and their host launchers.
// Each kernel is a thin grid over the stage tiles of mtp_device.hpp.
#include <algorithm>

#include "kernels.hpp"
#include "pm_tile.hpp"
#include "rollout_grid.hpp"
#include "wave_select.hpp"

namespace mtp {

__global__ __launch_bounds__(64) void k_set_ctrl(PlanDesc P, uint32_t r, int shift, const float* x0_src) {
  set_ctrl_block(P, r, shift, x0_src);
}

// One workgroup (the shift is in place through a scratch copy and a barrier);
// 1024 threads keep four times as many loads in flight as 256.
__global__ __launch_bounds__(1024) void k_shift(PlanDesc P) {
  shift_block<1024>(P, static_cast<int>(P.ctrl[1]));
}

__global__ __launch_bounds__(kCandThreads) void k_paths(PlanDesc P, int k) {
  __shared__ PathSmem sm;
  path_tile(P, P.ctrl[0], k, blockIdx.x, gridDim.x, sm);
}

static int cand_chunk(const PlanDesc& P) { return P.tc < kTChunk ? P.tc : kTChunk; }

// grid (candidate tiles, joints, horizon chunks of P.tc steps); LDS sized for
// the plan so that several workgroups fit on a compute unit
__global__ __launch_bounds__(kCandThreads) void k_candidates(PlanDesc P, int k) {
  extern __shared__ float cand_lds[];
  // tensor paths already drawn by the previous replan: only the local samples
  // and the nominal are written, and tiles of tensor paths alone return
  const bool ahead = P.cand_skip && P.ctrl[4] != 0u;
  const int b0 = static_cast<int>(blockIdx.x) * kCandThreads;
  if (ahead && b0 >= P.G - 1 && b0 + kCandThreads <= P.B - 1) return;
  const CandView v = cand_view_dyn(cand_lds, P.L, P.W, P.tc < kTChunk ? P.tc : kTChunk);
  const int t_begin = blockIdx.z * P.tc;
  cand_tile(P, P.ctrl[0], k, blockIdx.y, b0, t_begin, min(P.T, t_begin + P.tc), v, ahead ? kCandLocal : kCandAll);
}

__global__ __launch_bounds__(kTopkThreads) void k_entropy(PlanDesc P, int k) {
  __shared__ EntropySmem sm;
  entropy_block<kTopkThreads>(P, k, sm);
}

// Rollout workgroups are four waves: the waves of one workgroup go to the four
// SIMDs of a compute unit, while single-wave workgroups sharing a unit were seen
// to stack two waves on one SIMD now and then, doubling the time of a launch
// with fewer waves than SIMDs.
// Point mass: a workgroup rolls out a tile of kPmTileCands candidates
// (pm_tile.hpp).  Small launches are bound by the tile's latency (controls from
// memory, the two serial passes over the steps), large ones by the obstacle
// tests, which this form issues once per candidate and step.  Replan on eight
// lanes per candidate through the horizon before -> now: 3341 candidates x 77
// steps x 6 iterations 0.170 -> 0.158 ms; 15700 x 256 x 6 0.477 -> 0.414 ms.
// POINTS: see pm_tile_cost; a horizon of 16 or 32 steps fills one or two points of
// each thread, and testing the obstacles for the idle ones as well cost up to 6 %
// of a replan (12000 candidates x 16 steps, 30 obstacles).
constexpr int kPmTileCands = 16;
template <int POINTS>
__global__ __launch_bounds__(kRollThreads) void k_rollout_point_mass(PlanDesc P) {
  if (static_cast<int>(blockIdx.x) >= P.roll_blocks) { gen_tensor_tiles(P); return; }
  __shared__ PmTile<kPmTileCands> tile;
  __shared__ float4 obs[kMaxObstacles];
  const int tid = threadIdx.x;
  const int b0 = xcd_contiguous_block(blockIdx.x, P.roll_blocks) * kPmTileCands;
  const int n_pad = load_obstacles(P, obs);
  const size_t ld = static_cast<size_t>(P.ldU);
  // idle lanes of the last tile shadow the last candidate and store nothing
  const int c = tid % kPmTileCands, row = tid / kPmTileCands;
  const float* u = P.U + min(b0 + c, P.B - 1);
  constexpr int kRows = kRollThreads / kPmTileCands, kLoads = 2 * kTileSteps / kRows;
  const bool records = b0 < P.n_dbg;
  const float cost = pm_tile_cost<kPmTileCands, kRollThreads, POINTS>(
      P, tile, obs, n_pad,
      [&](int t0, int steps) {
        float v[kLoads];   // every load of the chunk in flight at once
#pragma unroll
        for (int i = 0; i < kLoads; ++i) v[i] = u[(2 * t0 + min(row + i * kRows, 2 * steps - 1)) * ld];
#pragma unroll
        for (int i = 0; i < kLoads; ++i) (&tile.u[0][0][0])[(row + i * kRows) * kPmTileCands + c] = v[i];
      },
      [&](int t, int dim, int cand, float pos, float vel) {
        if (records && b0 + cand < P.n_dbg) {
          const size_t ldx = static_cast<size_t>(P.n_dbg);
          P.X[(t * 4 + dim) * ldx + b0 + cand] = pos;
          P.X[(t * 4 + 2 + dim) * ldx + b0 + cand] = vel;
        }
      });
  if (tid < kPmTileCands && b0 + tid < P.B) P.cost[b0 + tid] = cost;
}

// Eight lanes per candidate through the horizon, each with an eighth of the
// obstacle table, for launches of more tiles than the chip holds at a time.
__global__ __launch_bounds__(kRollThreads) void k_rollout_point_mass_lanes(PlanDesc P) {
  __shared__ PointMassSmem sm;
  stage_obstacles(P, sm);
  __syncthreads();
  const int g = xcd_contiguous_block(blockIdx.x, P.roll_blocks) * kRollThreads + threadIdx.x;
  const int b = g / kPmLanes;
  if (b < P.B) rollout_point_mass_any<kPmLanes>(P, b, g % kPmLanes, sm);
}

// A compute unit holds four tiles.  Past that the last round of tiles leaves most
// of the chip idle, and short horizons pay the tile's serial passes for little;
// eight lanes per candidate are faster there, up to 32 obstacles (more do not fit
// their registers).  Over long horizons the tiles, which test every obstacle once,
// win again from seven per unit on, or with hardly any obstacle to test.  Replans of
// four iterations, tiles -> eight lanes: 18000 candidates x 20 steps, 30 obstacles
// 11 % shorter, 39000 x 20 14 %, 18000 x 50, 8 obstacles 4 %, 18000 x 200 2 to 5 %;
// 33000 x 200 1 % longer; 16000 x 50 12 % longer.
static_assert(kPmPoints<kPmTileCands, kRollThreads> == 4 && kPmTileCands * 16 == kRollThreads, "a point per 16 steps");
static_assert(kPmOverlapLanes == kPmLanes, "rollout_blocks counts the workgroups of the lanes");
static bool pm_on_lanes(const PlanDesc& P) {
  constexpr int kTilesPerUnit = 4, kManyTiles = 7, kLongHorizon = 64;
  const int tiles = (P.B + kPmTileCands - 1) / kPmTileCands, n_obs = (P.n_task - 6) / 3;
  return P.U2 == nullptr && n_obs <= 32 && tiles > kTilesPerUnit * P.gen_grid &&
         (P.T < kLongHorizon || (n_obs >= 8 && tiles <= kManyTiles * P.gen_grid));
}

template <int N, bool CONTACT, bool ONE>
__global__ __launch_bounds__(kRollThreads) MTP_ROLL_WAVES(ONE || N >= 20) void k_rollout_chain_pair(PlanDesc P) {
  if (static_cast<int>(blockIdx.x) >= P.roll_blocks) { gen_tensor_tiles(P); return; }
  const int g = xcd_contiguous_block(blockIdx.x, P.roll_blocks) * kRollThreads + threadIdx.x;
  const int b = g >> 1;
  if (b < P.B) rollout_chain_pair<N, CONTACT>(P, b, (g & 1) != 0);
}

// Tensor-path controls of iteration P.gen_k into P.U2 (P.roll_blocks = 0: every
// workgroup draws), run beside a time-sliced rollout that holds one wave per
// SIMD.  The launch asks for LDS that admits one of these workgroups per
// compute unit (one wave of 72 VGPRs per SIMD), so the rollout's workgroup
// (up to 440 registers per lane; 408 for 24 links with contact) finds its
// registers free on every unit whichever kernel is dispatched first.
__global__ __launch_bounds__(kCandThreads) void k_gen_tensor(PlanDesc P) { gen_tensor_tiles(P); }

// The small selection in a kernel of its own: beside the other it cost 1 us of it.
static TopkSizes topk_sizes(const PlanDesc& P) { return P.B <= kTopkBoundary ? kTopkSmall : kTopkLarge; }

template <TopkSizes SIZES>
__global__ __launch_bounds__(kTopkThreads) void k_topk(PlanDesc P) {
  __shared__ TopkSmem sm;
  topk_block<kTopkThreads, false, SIZES>(P, sm);
}

__global__ __launch_bounds__(kUpdThreads) void k_update(PlanDesc P) {
  const int o = blockIdx.x * (kUpdThreads / 64) + (threadIdx.x >> 6);
  // the last refit of a replan that drew the next replan's first tensor paths
  // (its launch follows the generator's): record the replan they are for
  if (P.gen_spec && blockIdx.x == 0 && threadIdx.x == 0) {
    P.ctrl[3] = P.ctrl[0] + 1u;
    P.ctrl[5] = 1u;
  }
  if (o < P.T * P.n) update_output(P, o);
}

// Refit of iteration k at the four steps t = 4 tq + c of joint j (one wave per
// step), and from each refitted (t, j) iteration k_next's local samples and
// nominal mean at (t, j) into P.U2 (its tensor paths were drawn during
// iteration k's rollout).  The four steps of a local sample come from one
// Philox block; every thread draws its first samples' normals while the waves
// refit.
__global__ __launch_bounds__(kUpdThreads) void k_update_next(PlanDesc P, int k_next) {
  __shared__ float mom[4][2];
  const int tq = static_cast<int>(blockIdx.x) / P.n, j = static_cast<int>(blockIdx.x) - tq * P.n;
  const int c = static_cast<int>(threadIdx.x) >> 6;
  const int t = 4 * tq + c;
  const uint32_t r = P.ctrl[0];
  float z[kLocalKeep][4];
  local_normals<kUpdThreads>(P, tq, j, k_next, r, z);
  if (t < P.T) {
    float mn, sn;
    update_output(P, t * P.n + j, &mn, &sn);
    if ((threadIdx.x & 63) == 0) { mom[c][0] = mn; mom[c][1] = sn; }
  }
  __syncthreads();
  local_store<kUpdThreads>(P, P.U2, tq, j, k_next, r, z, mom);
}

// The refit of iteration k from its elites' controls drawn again
// (regen_elites) rather than gathered from U, one workgroup per four steps of
// a joint; with NEXT also iteration k_next's local samples and nominal (as
// k_update_next), without it the last iteration's refit (as k_update, which
// also records the replan whose tensor paths were drawn when P.gen_spec).
template <bool NEXT>
__global__ __launch_bounds__(kUpdThreads) void k_refit_regen(PlanDesc P, int k, int k_next) {
  __shared__ RegenSmem sm;
  __shared__ float mom[4][2];
  const int tq = static_cast<int>(blockIdx.x) / P.n, j = static_cast<int>(blockIdx.x) - tq * P.n;
  const int c = static_cast<int>(threadIdx.x) >> 6;
  const int t = 4 * tq + c;
  const uint32_t r = P.ctrl[0];
  float z[kLocalKeep][4];
  if constexpr (NEXT) local_normals<kUpdThreads>(P, tq, j, k_next, r, z);
  if (!NEXT && P.gen_spec && blockIdx.x == 0 && threadIdx.x == 0) {
    P.ctrl[3] = P.ctrl[0] + 1u;
    P.ctrl[5] = 1u;
  }
  regen_elites(P, k, tq, j, sm);
  if (t < P.T) {
    float mn, sn;
    update_output_from(P, t * P.n + j, gptr(P.w), [&](int e) { return sm.vals[c][e]; }, &mn, &sn);
    if ((threadIdx.x & 63) == 0) { mom[c][0] = mn; mom[c][1] = sn; }
  }
  if constexpr (NEXT) {
    __syncthreads();
    local_store<kUpdThreads>(P, P.U2, tq, j, k_next, r, z, mom);
  }
}

// Top-E selection and refit of an iteration in one launch, one workgroup per
// four steps of a joint.  Every workgroup selects the elites for itself (the
// same values in each; the first stores them), then four of its waves refit one
// step each, as k_update, or k_update_next with NEXT.  The selection is one
// workgroup's latency either way, and one launch less is a microsecond per
// iteration.  Replans in two launches -> one (candidates x links x iterations):
// 9216 x 7 x 8 1.014 -> 0.994 ms; 3376 x 12 x 6 0.632 -> 0.621 ms; 3341 point
// masses x 6 157.7 -> 152.8 us; 13500 x 4 x 4 0.310 -> 0.303 ms.
constexpr int kFusedThreads = kTopkThreads;
template <bool NEXT, TopkSizes SIZES>
__global__ __launch_bounds__(kFusedThreads) void k_select_refit(PlanDesc P, int k_next) {
  __shared__ TopkSmem sm;
  __shared__ float mom[4][2];
  const int tq = static_cast<int>(blockIdx.x) / P.n, j = static_cast<int>(blockIdx.x) - tq * P.n;
  const int c = static_cast<int>(threadIdx.x) >> 6;
  const int t = 4 * tq + c;
  const uint32_t r = P.ctrl[0];
  float z[kLocalKeep][4];
  if constexpr (NEXT) local_normals<kFusedThreads>(P, tq, j, k_next, r, z);
  if (P.gen_spec && blockIdx.x == 0 && threadIdx.x == 0) {   // as k_update
    P.ctrl[3] = P.ctrl[0] + 1u;
    P.ctrl[5] = 1u;
  }
  topk_block<kFusedThreads, true, SIZES>(P, sm, blockIdx.x == 0);
  if (c < 4 && t < P.T) {
    const int o = t * P.n + j;
    const auto row = gptr(P.U) + static_cast<size_t>(o) * static_cast<size_t>(P.ldU);
    const float* w = topk_weights(sm);
    const int* elite = topk_elites(sm);
    float mn, sn;
    update_output_from(P, o, w, [&](int e) { return row[elite[e]]; }, &mn, &sn);
    if ((threadIdx.x & 63) == 0) { mom[c][0] = mn; mom[c][1] = sn; }
  }
  if constexpr (NEXT) {
    __syncthreads();
    local_store<kFusedThreads>(P, P.U2, tq, j, k_next, r, z, mom);
  }
}

// The same for few candidates and elites: one wave selects without barriers while
// the others draw their normals, in a workgroup of a refit tile's size.
constexpr int kSelectWave = kUpdThreads / 64 - 1;   // the wave with the fewest local samples to draw
template <bool NEXT>
__global__ __launch_bounds__(kUpdThreads) void k_select_refit_wave(PlanDesc P, int k_next) {
  __shared__ WaveSelectSmem sm;
  __shared__ int elite[64];
  __shared__ float weight[64];
  __shared__ float mom[4][2];
  const int tq = static_cast<int>(blockIdx.x) / P.n, j = static_cast<int>(blockIdx.x) - tq * P.n;
  const int c = static_cast<int>(threadIdx.x) >> 6, lane = threadIdx.x & 63;
  const int t = 4 * tq + c;
  const uint32_t r = P.ctrl[0];
  if (c == kSelectWave) {
    const auto cost = gptr(P.cost);
    float v[kWaveKeys];
    uint32_t o[kWaveKeys];
#pragma unroll
    for (int q = 0; q < kWaveKeys; ++q) v[q] = cost[min(lane + 64 * q, P.B - 1)];
#pragma unroll
    for (int q = 0; q < kWaveKeys; ++q) o[q] = lane + 64 * q < P.B ? cost_order(v[q]) : 0xFFFFFFFFu;
    // as topk_block: the values that an image does not give back are read again
    const WaveElite el = wave_elites(o, lane, P.B, P.E, P.lam, sm, [&](int idx, float v) {
      return (v == 0.0f || v == INFINITY) ? cost[idx] : v;
    });
    if (lane < P.E) {
      elite[lane] = el.idx;
      weight[lane] = el.weight;
      if (blockIdx.x == 0) {
        gptr(P.eidx)[lane] = el.idx;
        gptr(P.ecost)[lane] = el.cost;
        gptr(P.w)[lane] = el.weight;
        if (lane == 0 && !(el.best < INFINITY)) atomicOr(&P.ctrl[2], 1u);
      }
    }
  }
  float z[kLocalKeep][4];
  if constexpr (NEXT) local_normals<kUpdThreads>(P, tq, j, k_next, r, z);
  if (P.gen_spec && blockIdx.x == 0 && threadIdx.x == 0) {   // as k_update
    P.ctrl[3] = P.ctrl[0] + 1u;
    P.ctrl[5] = 1u;
  }
  __syncthreads();
  if (t < P.T) {
    const int o = t * P.n + j;
    const auto row = gptr(P.U) + static_cast<size_t>(o) * static_cast<size_t>(P.ldU);
    float mn, sn;
    update_output_from(P, o, weight, [&](int e) { return row[elite[e]]; }, &mn, &sn);
    if (lane == 0) { mom[c][0] = mn; mom[c][1] = sn; }
  }
  if constexpr (NEXT) {
    __syncthreads();
    local_store<kUpdThreads>(P, P.U2, tq, j, k_next, r, z, mom);
  }
}

// ---------------------------------------------------------------- dispatch

static const int kChainLinks[] = {
#define X(N) N,
    MTP_CHAIN_LINKS(X)
#undef X
};
static const int kContactLinks[] = {
#define X(N) N,
    MTP_CONTACT_LINKS(X)
#undef X
};

bool rollout_supported(int dyn, int n_links) {
  if (dyn == kPointMass) return true;
  const int* tab = dyn == kChain ? kChainLinks : kContactLinks;
  const int cnt = dyn == kChain ? int(sizeof(kChainLinks) / sizeof(int)) : int(sizeof(kContactLinks) / sizeof(int));
  for (int i = 0; i < cnt; ++i)
    if (tab[i] == n_links) return true;
  return false;
}

int supported_chain_links(int* out, int cap) {
  const int cnt = int(sizeof(kChainLinks) / sizeof(int));
  for (int i = 0; i < cnt && i < cap; ++i) out[i] = kChainLinks[i];
  return cnt;
}

// Workgroups of a rollout on one to four lanes per candidate (eight for the
// point mass): what the decision to draw ahead goes by.  The point mass and the
// wide forms launch more.
int rollout_blocks(const PlanDesc& P) {
  const long long lanes_per = P.dyn == kPointMass             ? kPmOverlapLanes
                              : is_quad_chain(P.dyn, P.n_links) ? 4
                              : is_pair_chain(P.dyn, P.n_links) ? 2
                                                                : 1;
  return static_cast<int>((lanes_per * P.B + kRollThreads - 1) / kRollThreads);
}

// LDS that leaves room for only one workgroup per compute unit (160 KB each).
// A rollout launch with fewer workgroups than units asks for it so that no two
// of its workgroups, or a rollout and a generator workgroup, share a unit and
// its SIMDs (the dispatcher was seen to pair workgroups on a unit now and
// then, which doubles those waves' time).
constexpr size_t kOnePerUnitLds = 96 * 1024;

// LDS of a rollout launch that also draws tensor-path controls: the candidate
// tile's arrays over the whole horizon, at least kOnePerUnitLds.
static size_t gen_tile_bytes(const PlanDesc& P) {
  return sizeof(float) * static_cast<size_t>(cand_dyn_floats(P.L, P.W, P.T < kTChunk ? P.T : kTChunk));
}
static size_t gen_lds_bytes(const PlanDesc& P) { return std::max(gen_tile_bytes(P), kOnePerUnitLds); }

template <bool ONE>
static hipError_t launch_rollout_kernel(const PlanDesc& P, dim3 grid, size_t lds, hipStream_t st);

// The rollout of P.U; with gen_k >= 0 the launch adds workgroups that draw
// iteration gen_k's tensor-path controls into P.U2.
static hipError_t launch_rollout(const PlanDesc& P0, hipStream_t st, int gen_k) {
  PlanDesc P = P0;
  if (is_pair_chain(P.dyn, P.n_links) && P.seg_ctl != nullptr && P.seg_grid > 0) return launch_rollout_seg(P, st);
  const bool gen = gen_k >= 0 && P.U2 != nullptr;
  const int lanes = wide_lanes(P, gen);
  const bool tiled = P.dyn == kPointMass && !pm_on_lanes(P);
  P.roll_blocks = lanes > 0 ? wide_blocks(P, lanes)
                  : tiled   ? (P.B + kPmTileCands - 1) / kPmTileCands
                            : rollout_blocks(P);
  P.gen_k = gen_k;
  int blocks = P.roll_blocks;
  size_t lds = 0;
  if (gen) {
    // the units that the rollout's last round leaves
    int gens = std::max(P.gen_grid - P.roll_blocks % P.gen_grid, kMinGenBlocks);
    // A point mass's tiles share units with each other and with the generator:
    // where they leave too few of their own, the generator takes the eight-lane
    // form's share (5000 candidates x 64 steps, four iterations: 164 us with 32
    // workgroups drawing, 119 with 99).
    if (tiled && P.roll_blocks + kMinGenBlocks > P.gen_grid)
      gens = std::max(P.gen_grid - rollout_blocks(P), kMinGenBlocks);
    blocks = P.roll_blocks + gens;
    lds = blocks <= P.gen_grid ? gen_lds_bytes(P) : gen_tile_bytes(P);
  } else if (P.roll_blocks <= P.gen_grid) {
    lds = kOnePerUnitLds;
  }
  const dim3 grid(blocks);
  if (lanes > 0) return launch_rollout_wide(P, lanes, grid, lds, st, blocks <= P.gen_grid);
  return blocks <= P.gen_grid ? launch_rollout_kernel<true>(P, grid, lds, st)
                              : launch_rollout_kernel<false>(P, grid, lds, st);
}

template <bool ONE>
static hipError_t launch_rollout_kernel(const PlanDesc& P, dim3 grid, size_t lds, hipStream_t st) {
  if (P.dyn == kPointMass) {
    if (pm_on_lanes(P)) k_rollout_point_mass_lanes<<<grid, kRollThreads, lds, st>>>(P);
    else if (P.T <= 16) k_rollout_point_mass<1><<<grid, kRollThreads, lds, st>>>(P);
    else if (P.T <= 32) k_rollout_point_mass<2><<<grid, kRollThreads, lds, st>>>(P);
    else k_rollout_point_mass<4><<<grid, kRollThreads, lds, st>>>(P);
    return hipGetLastError();
  }
  if (is_quad_chain(P.dyn, P.n_links)) return launch_rollout_quad(P, grid, lds, st, ONE);
  if (is_pair_chain(P.dyn, P.n_links)) {
    if (P.dyn == kChain) {
      switch (P.n_links) {
#define X(N) case N: if constexpr (pair_chain_links<N>()) { k_rollout_chain_pair<N, false, ONE><<<grid, kRollThreads, lds, st>>>(P); return hipGetLastError(); } break;
        MTP_CHAIN_LINKS(X)
#undef X
        default: break;
      }
    } else {
      switch (P.n_links) {
#define X(N) case N: if constexpr (pair_chain_links<N>()) { k_rollout_chain_pair<N, true, ONE><<<grid, kRollThreads, lds, st>>>(P); return hipGetLastError(); } break;
        MTP_CONTACT_LINKS(X)
#undef X
        default: break;
      }
    }
    return hipErrorInvalidValue;
  }
  if (P.dyn == kChain) {
    // Two and three links: the rollout is shorter under this unit's option, the
    // generator under the other's.  Rollouts alone, us here and there: 3 links, 250
    // candidates x 96 steps 80.0 and 81.8, 40000 x 64 55.9 and 56.5; 2 links, 1100 x
    // 50 31.2 and 32.3, 20000 x 64 40.8 and 40.0.  Replans of four iterations with
    // the generator, 3 links, 600 x 32 154.4 and 152.5, 39000 x 16 260 and 250, 20000
    // x 256 990 and 1015, but 55000 x 300, as long as its generator, 1539 and 1138; 2
    // links, 73 x 200, five iterations 592 and 612.
    const bool alone = static_cast<int>(grid.x) == P.roll_blocks;
    const bool bound = !alone && gen_us(P, static_cast<int>(grid.x) - P.roll_blocks) > narrow_wave_us(P);
    const bool here = P.n_links <= 3 && (P.n_links == 3 || P.B <= 8192) && (alone || (P.T >= 96 && !bound));
    if (!here) return launch_rollout_line(P, grid, lds, st);
    switch (P.n_links) {
#define X(N) case N: if constexpr (N <= 3) { k_rollout_chain<N, false, ONE><<<grid, kRollThreads, lds, st>>>(P); return hipGetLastError(); } break;
      MTP_CHAIN_LINKS(X)
#undef X
      default: break;
    }
    return hipErrorInvalidValue;
  }
  switch (P.n_links) {
#define X(N) case N: if constexpr (!pair_chain_links<N>()) { k_rollout_chain<N, true, ONE><<<grid, kRollThreads, lds, st>>>(P); return hipGetLastError(); } break;
    MTP_CONTACT_LINKS(X)
#undef X
    default: break;
  }
  return hipErrorInvalidValue;
}

static hipError_t launch_candidates(const PlanDesc& P, int k, hipStream_t st) {
  if (P.P > 0 && P.wor) {
    k_paths<<<(P.P + kCandThreads - 1) / kCandThreads, kCandThreads, 0, st>>>(P, k);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const dim3 grid((P.B + kCandThreads - 1) / kCandThreads, P.n, (P.T + P.tc - 1) / P.tc);
  const size_t lds = sizeof(float) * static_cast<size_t>(cand_dyn_floats(P.L, P.W, cand_chunk(P)));
  k_candidates<<<grid, kCandThreads, lds, st>>>(P, k);
  return hipGetLastError();
}

hipError_t launch_set_ctrl(const PlanDesc& P, uint32_t r, int shift, const float* x0_src, hipStream_t st) {
  k_set_ctrl<<<1, 64, 0, st>>>(P, r, shift, x0_src);
  return hipGetLastError();
}

hipError_t launch_shift(const PlanDesc& P, hipStream_t st) {
  k_shift<<<1, 1024, 0, st>>>(P);
  return hipGetLastError();
}

hipError_t launch_stage(const PlanDesc& P, int stage, int k, hipStream_t st) {
  switch (stage) {
    case 0:
      return launch_candidates(P, k, st);
    case 1:
      return launch_rollout(P, st, -1);
    case 2:
      if (topk_sizes(P) == kTopkSmall) k_topk<kTopkSmall><<<1, kTopkThreads, 0, st>>>(P);
      else k_topk<kTopkLarge><<<1, kTopkThreads, 0, st>>>(P);
      if (P.diag & 1) {
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        k_entropy<<<1, kTopkThreads, 0, st>>>(P, k);
      }
      return hipGetLastError();
    case 3: {
      const int outs = P.T * P.n;
      const int per = kUpdThreads / 64;
      k_update<<<(outs + per - 1) / per, kUpdThreads, 0, st>>>(P);
      return hipGetLastError();
    }
    default:
      return hipErrorInvalidValue;
  }
}

static bool is_sliced(const PlanDesc& P) {
  return is_pair_chain(P.dyn, P.n_links) && P.seg_ctl != nullptr && P.seg_grid > 0;
}

// the plan's layout assumed a 256-unit chip; a device without a free unit
// beyond the rollout's workgroups runs the plain sequence
static bool draws_ahead(const PlanDesc& P) {
  return P.U2 != nullptr && (is_sliced(P) || P.gen_grid > rollout_blocks(P));
}

// Stage `stage` of iteration k within a run of iterations [k0, k1).  With the
// overlap (P.U2 set) iteration k works on U (k1 - 1 - k even, so the last
// iteration always ends in U) or U2 (odd); its rollout also draws iteration
// k+1's tensor-path controls into the other buffer on the compute units the
// rollout leaves idle, and its refit writes iteration k+1's local samples and
// nominal mean there from each refitted (t, j), so iteration k+1 launches no
// candidate kernel.  The values are those of the plain sequence: the tensor
// paths do not depend on the sampling distribution.
hipError_t launch_iteration_stage(const PlanDesc& P, int stage, int k, int k0, int k1, hipStream_t st,
                                  const SideLane* side) {
  if (!draws_ahead(P)) return launch_stage(P, stage, k, st);
  const bool sliced = is_sliced(P);
  PlanDesc Pk = P;
  if ((k1 - 1 - k) & 1) { Pk.U = P.U2; Pk.U2 = P.U; }
  // a whole replan of a plan that draws across replans: iteration 0 may take
  // the tensor paths the previous replan drew, and the last iteration draws
  // the next replan's into the buffer iteration 0 reads (the other one, K even)
  const bool across = P.spec && k0 == 0 && k1 == P.K;
  const bool last = k + 1 >= k1;
  switch (stage) {
    case 0:
      if (k > k0) return hipSuccess;
      Pk.cand_skip = across ? 1 : 0;
      return launch_candidates(Pk, k, st);
    case 1: {
      if (last && !across) return launch_rollout(Pk, st, -1);
      hipError_t e = hipSuccess;
      if (!sliced) {
        Pk.gen_spec = last ? 1 : 0;
        return launch_rollout(Pk, st, last ? 0 : k + 1);
      }
      PlanDesc G = Pk;
      G.roll_blocks = 0;
      G.gen_k = last ? 0 : k + 1;
      G.gen_spec = last ? 1 : 0;
      const size_t tile = sizeof(float) * static_cast<size_t>(cand_dyn_floats(P.L, P.W, P.T < kTChunk ? P.T : kTChunk));
      const size_t lds = seg_lds_bytes(P) > 0 ? tile : std::max(tile, kOnePerUnitLds);
      const hipStream_t gs = side != nullptr ? side->st : st;
      if (side != nullptr) {
        e = hipEventRecord(side->fork, st);
        if (e == hipSuccess) e = hipStreamWaitEvent(side->st, side->fork, 0);
        if (e != hipSuccess) return e;
        k_gen_tensor<<<G.gen_grid, kCandThreads, lds, gs>>>(G);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
      }
      e = launch_rollout(Pk, st, -1);
      if (e != hipSuccess) return e;
      if (side == nullptr) {
        k_gen_tensor<<<G.gen_grid, kCandThreads, lds, gs>>>(G);
        return hipGetLastError();
      }
      e = hipEventRecord(side->join, side->st);
      if (e == hipSuccess) e = hipStreamWaitEvent(st, side->join, 0);
      return e;
    }
    case 3: {
      const bool regen = refit_regenerates(Pk.interp, Pk.p, Pk.wor, Pk.E, Pk.B);
      const int tiles = ((Pk.T + 3) / 4) * Pk.n;
      if (last) {
        // the last refit also records the replan whose tensor paths were drawn
        Pk.gen_spec = across ? 1 : 0;
        if (!regen) return launch_stage(Pk, stage, k, st);
        k_refit_regen<false><<<tiles, kUpdThreads, 0, st>>>(Pk, k, -1);
        return hipGetLastError();
      }
      if (regen) k_refit_regen<true><<<tiles, kUpdThreads, 0, st>>>(Pk, k, k + 1);
      else k_update_next<<<tiles, kUpdThreads, 0, st>>>(Pk, k + 1);
      return hipGetLastError();
    }
    default: return launch_stage(Pk, stage, k, st);
  }
}

// Stages 2 and 3 of iteration k in one launch where every workgroup of
// k_select_refit has a compute unit of its own (its LDS admits one per unit, so a
// second round would select once more) and the costs fit that LDS.
static bool fuses_refit(const PlanDesc& P) {
  return (P.diag & 1) == 0 && P.B <= kTopkCache && ((P.T + 3) / 4) * P.n <= P.gen_grid &&
         !refit_regenerates(P.interp, P.p, P.wor, P.E, P.B);
}

// By one wave where it holds every cost in its registers and an elite per lane,
// on up to four of its small workgroups per compute unit.  Replans on the
// 1024-thread selection (or its two launches) -> by one wave: 561 candidates x 3
// links x 4 iterations 162.3 -> 152.6 us; 780 point masses x 6 140.4 -> 124.4 us;
// 900 x 7 x 6 422 -> 406 us; 900 x 12 x 128 steps x 6 (384 tiles) 1057 -> 1034 us.
// Not where the elites are a good part of the candidates: the short list that the
// wave orders overflows then (64 of 128 candidates: a microsecond more an iteration).
static bool selects_by_wave(const PlanDesc& P) {
  return (P.diag & 1) == 0 && P.B <= 64 * kWaveKeys && P.E <= 64 && 4 * P.E <= P.B &&
         ((P.T + 3) / 4) * P.n <= 4 * P.gen_grid;
}

hipError_t launch_iteration(const PlanDesc& P, int k, int k0, int k1, hipStream_t st, const SideLane* side) {
  const bool by_wave = selects_by_wave(P), fused = by_wave || fuses_refit(P);
  for (int stage = 0; stage < (fused ? 2 : 4); ++stage) {
    const hipError_t e = launch_iteration_stage(P, stage, k, k0, k1, st, side);
    if (e != hipSuccess) return e;
  }
  if (!fused) return hipSuccess;
  const bool ahead = draws_ahead(P), last = k + 1 >= k1;
  PlanDesc Pk = P;
  if (ahead && ((k1 - 1 - k) & 1)) { Pk.U = P.U2; Pk.U2 = P.U; }
  Pk.gen_spec = (ahead && last && P.spec && k0 == 0 && k1 == P.K) ? 1 : 0;
  const int tiles = ((P.T + 3) / 4) * P.n;
  if (by_wave) {
    if (ahead && !last) k_select_refit_wave<true><<<tiles, kUpdThreads, 0, st>>>(Pk, k + 1);
    else k_select_refit_wave<false><<<tiles, kUpdThreads, 0, st>>>(Pk, -1);
  } else if (topk_sizes(P) == kTopkSmall) {
    if (ahead && !last) k_select_refit<true, kTopkSmall><<<tiles, kFusedThreads, 0, st>>>(Pk, k + 1);
    else k_select_refit<false, kTopkSmall><<<tiles, kFusedThreads, 0, st>>>(Pk, -1);
  } else {
    if (ahead && !last) k_select_refit<true, kTopkLarge><<<tiles, kFusedThreads, 0, st>>>(Pk, k + 1);
    else k_select_refit<false, kTopkLarge><<<tiles, kFusedThreads, 0, st>>>(Pk, -1);
  }
  return hipGetLastError();
}

hipError_t gen_configure(PlanDesc* P) {
  int dev = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  P->gen_grid = cus;
  return hipSuccess;
}

}  // namespace mtp
