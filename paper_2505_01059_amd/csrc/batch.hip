// Persistent batched execution of many MTP instances in one launch.
//
// Work is cut into items (instance, phase, iteration, tile).  A fixed grid of
// workgroups loops: take the next queue position with an atomic counter, wait
// until that position has been published, run the tile, and count it done for
// its instance.  The workgroup that finishes the last tile of an instance's
// phase publishes the tiles of that instance's next phase at the queue's tail.
// Positions are taken in order and every item is published by a tile that sat
// at a lower position, so the lowest unfinished position never waits on work
// behind it: the loop drains without any co-residency assumption.  Every wait
// is bounded by a wall-clock limit; a timeout raises an error flag that makes
// all workgroups leave, so the grid always terminates.
//
// Per-instance stages run the same tile functions as the single-plan kernels,
// and every reduction has an order fixed by the instance alone, so a result
// does not depend on which workgroup ran which tile or on the other instances.
#define MTP_SHARED_LAUNCH 1   // items read what others of the launch stored
#include "batch.hpp"
#include "batch_cand.hpp"
#include "rollout_wide.hpp"

namespace mtp {

__device__ __forceinline__ uint32_t phase_tiles(const PlanDesc& P, uint32_t phase, uint32_t shape) {
  return phase_items(P.B, P.P, P.T, P.n, phase, is_quad_chain(P.dyn, P.n_links), is_pair_chain(P.dyn, P.n_links),
                     P.wor != 0, shape);
}

union BatchSmem {
  PathSmem path;
  BatchCandSmem cand;
  TopkSmem topk;
  EntropySmem ent;
};

struct BatchShared {
  BatchItem item;
  uint32_t pos;
  uint32_t pub_pos, pub_count, pub_phase, pub_k;
  int32_t publish;
  int32_t abort;
  int32_t acquire;  // the item's inputs may be newer than the caches
  uint32_t fresh;   // positions whose items' inputs are not
};

// Queue words travel at agent scope, past the XCDs' L2s.
__device__ __forceinline__ uint32_t load_agent(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

static_assert(sizeof(BatchItem) == 16, "two 64-bit words");
__device__ __forceinline__ void store_item(BatchItem* p, const BatchItem& it) {
  uint64_t* w = reinterpret_cast<uint64_t*>(p);
  store_agent(w, static_cast<uint64_t>(it.phase) << 32 | it.inst);
  store_agent(w + 1, static_cast<uint64_t>(it.tile) << 32 | it.k);
}

__device__ __forceinline__ BatchItem load_item(const BatchItem* p) {
  const uint64_t* w = reinterpret_cast<const uint64_t*>(p);
  const uint64_t a = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint64_t b = __hip_atomic_load(w + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  BatchItem it;
  it.inst = static_cast<uint32_t>(a); it.phase = static_cast<uint32_t>(a >> 32);
  it.k = static_cast<uint32_t>(b); it.tile = static_cast<uint32_t>(b >> 32);
  return it;
}

// One rollout tile of each form, out of line (the descriptor is read again from
// its uniform address).  Inlined into the one persistent kernel, the forms
// shared a single register allocation, so that a change in one of them moved
// the others' times by 3 to 5 %, and more forms did not fit: 256 uneven
// instances 82.0 ms per replan inlined, 81.6 ms out of line.
__device__ __forceinline__ PlanDesc load_desc(const PlanDesc* desc) {
  const uint64_t a = reinterpret_cast<uint64_t>(desc);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a >> 32));
  return *reinterpret_cast<const PlanDesc*>(static_cast<uint64_t>(hi) << 32 | lo);
}

template <int N, bool CONTACT, bool EQ>
__device__ __noinline__ void roll_chain_tile(const PlanDesc* desc, uint32_t tile) {
  const PlanDesc P = load_desc(desc);
  tile = __builtin_amdgcn_readfirstlane(tile);
  const int t = static_cast<int>(threadIdx.x);
  if constexpr (!CONTACT && quad_chain_links<N>()) {
    const int b = static_cast<int>(tile) * (kBatchThreads / 4) + (t >> 2);
    if (b < P.B) rollout_chain_quad<N>(P, b, t & 3);
  } else if constexpr (pair_chain_links<N>()) {
    const int b = static_cast<int>(tile) * (kBatchThreads / 2) + (t >> 1);
    if (b < P.B) rollout_chain_pair<N, CONTACT, EQ>(P, b, (t & 1) != 0);
  } else {
    const int b = static_cast<int>(tile) * kBatchThreads + t;
    if (b < P.B) rollout_chain<N, CONTACT>(P, b);
  }
}

// The same tile on a wide form, 2^LG times the narrow lanes per candidate.
template <int N, bool CONTACT, bool EQ, int LG>
__device__ __noinline__ void roll_wide_tile(const PlanDesc* desc, uint32_t tile) {
  const PlanDesc P = load_desc(desc);
  tile = __builtin_amdgcn_readfirstlane(tile);
  constexpr bool kPair = pair_chain_links<N>();
  constexpr int kLanes = (kPair ? 2 : 1) << LG;
  constexpr int kWriter = kPair ? kLanes / 2 - 1 : kLanes - 1;
  const int t = static_cast<int>(threadIdx.x), pos = t % kLanes;
  const int bb = static_cast<int>(tile) * (kBatchThreads / kLanes) + t / kLanes;
  const bool live = bb < P.B;
  const int b = live ? bb : P.B - 1;   // idle groups shadow the last candidate and store nothing
  float total = 0.0f;
  for (int rep = 0; rep < P.R; ++rep) {
    if constexpr (kPair) total += rollout_half<N, (1 << LG), CONTACT, EQ>(P, b, pos, rep, live);
    else total += rollout_line<N, kLanes, CONTACT>(P, b, pos, rep, live);
  }
  if (live && pos == kWriter) store_result(&P.cost[b], finite_or_inf(P.R == 1 ? total : total / static_cast<float>(P.R)));
}

template <int N, bool CONTACT>
__device__ __forceinline__ void roll_chain(const PlanDesc* desc, bool eq, uint32_t lg, uint32_t tile) {
  constexpr uint32_t kMaxLg = max_wide_lg(CONTACT ? kChainContact : kChain, N);
  if constexpr (pair_chain_links<N>()) {
    if constexpr (kMaxLg >= 1) {
      if (lg == 1u) {
        if (eq) roll_wide_tile<N, CONTACT, true, 1>(desc, tile);
        else roll_wide_tile<N, CONTACT, false, 1>(desc, tile);
        return;
      }
    }
    if constexpr (kMaxLg >= 2) {
      if (lg == 2u) {
        if (eq) roll_wide_tile<N, CONTACT, true, 2>(desc, tile);
        else roll_wide_tile<N, CONTACT, false, 2>(desc, tile);
        return;
      }
    }
    // In contact, links of one length take the per-link form as well: with the
    // length held once the allocator spills in every solver stage of 24 links
    // (69632 candidates x 256 steps: 26.3 ms per iteration, per link 5.3).
    if (!CONTACT && eq) roll_chain_tile<N, CONTACT, !CONTACT>(desc, tile);
    else roll_chain_tile<N, CONTACT, false>(desc, tile);
  } else {
    if constexpr (kMaxLg >= 2) {
      if (lg == 1u) { roll_wide_tile<N, CONTACT, false, 1>(desc, tile); return; }
      if (lg == 2u) { roll_wide_tile<N, CONTACT, false, 2>(desc, tile); return; }
    }
    roll_chain_tile<N, CONTACT, false>(desc, tile);
  }
}

__device__ __noinline__ void roll_point_mass_tile(const PlanDesc* desc, uint32_t tile) {
  __shared__ PointMassSmem pm;
  const PlanDesc P = load_desc(desc);
  const int b = static_cast<int>(__builtin_amdgcn_readfirstlane(tile)) * kBatchThreads + static_cast<int>(threadIdx.x);
  stage_obstacles(P, pm);
  __syncthreads();
  if (b < P.B) rollout_point_mass_any(P, b, 0, pm);
}

__device__ __forceinline__ void run_rollout_tile(const PlanDesc* desc, const PlanDesc& P, uint32_t lg, uint32_t tile) {
  if (P.dyn == kPointMass) { roll_point_mass_tile(desc, tile); return; }
  const bool eq = P.eq_len != 0;
  if (P.dyn == kChain) {
    switch (P.n_links) {
#define X(N) case N: roll_chain<N, false>(desc, eq, lg, tile); return;
      MTP_CHAIN_LINKS(X)
#undef X
      default: return;
    }
  }
  switch (P.n_links) {
#define X(N) case N: roll_chain<N, true>(desc, eq, lg, tile); return;
    MTP_CONTACT_LINKS(X)
#undef X
    default: return;
  }
}

// Refit of the outputs [base, base + per) an item holds, the waves taking kRefits
// at a time: the elites' indices and weights are read once for them and their
// gathers from U are in flight together (an output alone waits for its indices,
// then for its gather; replans of 256 uneven instances 74.9 -> 71.9 ms, of 32 9.9
// -> 9.6).  For elite sets that update_output keeps in registers.
constexpr int kRefits = 4;
__device__ __noinline__ void refit_tile(const PlanDesc* desc, int base, int per) {
  const PlanDesc P = load_desc(desc);
  base = __builtin_amdgcn_readfirstlane(base);
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6), lane = threadIdx.x & 63;
  const int end = min(base + __builtin_amdgcn_readfirstlane(per), P.T * P.n);
  constexpr int kWaves = kBatchThreads / 64;
  int idx[kUpdKeep];
  float w[kUpdKeep];
#pragma unroll
  for (int q = 0; q < kUpdKeep; ++q) {
    const int e = min(lane + 64 * q, P.E - 1);
    if (64 * q < P.E) {
      idx[q] = gptr(P.eidx)[e];
      w[q] = gptr(P.w)[e];
    }
  }
  const size_t ld = static_cast<size_t>(P.ldU);
  for (int o0 = base + wave * kRefits; o0 < end; o0 += kWaves * kRefits) {
    float keep[kRefits][kUpdKeep], m[kRefits], v[kRefits], mu_old[kRefits], sg_old[kRefits];
#pragma unroll
    for (int i = 0; i < kRefits; ++i) {
      const int o = min(o0 + i, end - 1);
      const auto row = gptr(P.U) + static_cast<size_t>(o) * ld;
      mu_old[i] = gptr(P.mu)[o];
      sg_old[i] = gptr(P.sigma)[o];
#pragma unroll
      for (int q = 0; q < kUpdKeep; ++q)
        if (64 * q < P.E) keep[i][q] = row[idx[q]];
    }
    // the sums of update_output_from
#pragma unroll
    for (int i = 0; i < kRefits; ++i) {
      m[i] = 0.0f;
#pragma unroll
      for (int q = 0; q < kUpdKeep; ++q)
        if (lane + 64 * q < P.E) m[i] = fmaf(w[q], keep[i][q], m[i]);
      m[i] = wave_sum64(m[i]);
    }
#pragma unroll
    for (int i = 0; i < kRefits; ++i) {
      v[i] = 0.0f;
#pragma unroll
      for (int q = 0; q < kUpdKeep; ++q)
        if (lane + 64 * q < P.E) {
          const float dv = keep[i][q] - m[i];
          v[i] = fmaf(w[q], dv * dv, v[i]);
        }
      v[i] = wave_sum64(v[i]);
    }
#pragma unroll
    for (int i = 0; i < kRefits; ++i) {
      const int o = o0 + i;
      const float sd = fmaxf(sqrtf(v[i]), P.sigma_min);
      const float mn = fmaf(P.alpha, mu_old[i] - m[i], m[i]);
      const float sn = fmaf(P.alpha, sg_old[i] - sd, sd);
      if (lane == 0 && o < end) {
        store_result(&P.mu[o], mn);
        store_result(&P.sigma[o], sn);
        if (o < P.n) store_result(&P.action[o], keep[i][0]);
      }
    }
  }
}

#ifndef MTP_BATCH_MIN_WG_PER_CU
#define MTP_BATCH_MIN_WG_PER_CU 1
#endif

__global__ __launch_bounds__(kBatchThreads, MTP_BATCH_MIN_WG_PER_CU) void k_batch_persistent(const PlanDesc* __restrict__ descs,
                                                                    InstCtl* __restrict__ ictl, BatchCtl* ctl,
                                                                    BatchItem* __restrict__ queue,
                                                                    uint32_t* __restrict__ ready,
                                                                    uint64_t wait_ticks) {
  __shared__ BatchSmem sm;
  __shared__ BatchShared sh;
  const int tid = threadIdx.x;
  const uint32_t epoch = ctl->epoch;
  const uint32_t total = ctl->total;
  if (tid == 0) sh.fresh = 0u;
  // rollout items of several tiles run one tile per pass of this loop: `sub`
  // is the tile of the current item to run next (0: take a new item)
  uint32_t sub = 0;
  for (;;) {
    if (sub == 0u) {
      if (tid == 0) {
        sh.pos = atomicAdd(&ctl->head, 1u);
        sh.abort = 0;
      }
      __syncthreads();
      const uint32_t pos = sh.pos;
      if (pos >= total) break;
      if (tid == 0) {
        const uint64_t t0 = wall_clock64();
        uint32_t polls = 0u;
        while (load_agent(&ready[pos]) != epoch) {
          if ((++polls & 15u) == 0u && (load_agent(&ctl->error) != 0u || wall_clock64() - t0 > wait_ticks)) {
            atomicOr(&ctl->error, 1u);
            sh.abort = 1;
            break;
          }
          __builtin_amdgcn_s_sleep(2);
        }
        if (!sh.abort) sh.item = load_item(&queue[pos]);
        sh.acquire = pos >= sh.fresh;
        if (sh.acquire) sh.fresh = load_agent(&ctl->tail);
      }
      __syncthreads();
      if (sh.abort) break;
      // Acquire (an invalidation, no write-back).  An item's inputs reached memory
      // before its position was taken from the tail, so one invalidation serves
      // every position below the tail read before it: under load most items need
      // none.
      if (sh.acquire) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    const uint32_t inst = __builtin_amdgcn_readfirstlane(sh.item.inst);
    const uint32_t phase_word = __builtin_amdgcn_readfirstlane(sh.item.phase);
    const uint32_t phase = phase_word & kItemPhaseMask;
    const uint32_t shape = phase_word >> kItemShapeShift;   // the instance's item shape, carried by its items
    const uint32_t k = __builtin_amdgcn_readfirstlane(sh.item.k);
    const uint32_t tile = __builtin_amdgcn_readfirstlane(sh.item.tile);
    const PlanDesc P = descs[inst];

    switch (phase) {
      case kPhShift:
        shift_block<kBatchThreads>(P, static_cast<int>(P.ctrl[1]));
        break;
      case kPhPaths:
        path_tile(P, P.ctrl[0], static_cast<int>(k), static_cast<int>(tile), static_cast<int>(phase_tiles(P, kPhPaths, shape)),
                  sm.path);
        break;
      case kPhCand: {
        // an item is 2^cand_lg consecutive candidate tiles with all their
        // joints, or one joint of them
        const uint32_t r = P.ctrl[0];
        const bool one_joint = shape_cand_joint(shape) != 0u;
        const int group = one_joint ? static_cast<int>(tile) / P.n : static_cast<int>(tile);
        const int j0 = one_joint ? static_cast<int>(tile) - group * P.n : 0;
        const int j1 = one_joint ? j0 + 1 : P.n;
        const int per = 1 << shape_cand_lg(shape);
        const int n_tiles = (P.B + kCandThreads - 1) / kCandThreads;
        const int ct1 = min(group * per + per, n_tiles);
        for (int ct = group * per; ct < ct1; ++ct) {
          batch_cand_tile(P, r, static_cast<int>(k), j0, j1, ct * kCandThreads, sm.cand);
          __syncthreads();
        }
        break;
      }
      case kPhRoll:
        // an item is 2^roll_lg consecutive rollout tiles, one per pass
        run_rollout_tile(descs + inst, P, shape_wide_lg(shape), (tile << shape_roll_lg(shape)) + sub);
        break;
      case kPhTopk:
        topk_block<kBatchThreads>(P, sm.topk);
        if (P.diag & 1) {
          __syncthreads();
          entropy_block<kBatchThreads>(P, static_cast<int>(k), sm.ent);
        }
        break;
      default: {
        // few outputs: one per wave, here (the tile out of line costs them 1 %)
        const int per = 1 << shape_upd_lg(shape), base = static_cast<int>(tile) * per;
        if (per >= kRefits * (kBatchThreads / 64) && P.E <= 64 * kUpdKeep) {
          refit_tile(descs + inst, base, per);
        } else {
          for (int m = tid >> 6; m < per; m += kBatchThreads / 64)
            if (base + m < P.T * P.n) update_output(P, base + m);
        }
        break;
      }
    }
    // Candidate, rollout and refit items store everything at agent scope (another
    // XCD reads it, or writes it again in the next iteration): waiting for the
    // stores releases it.  The others' results, and recorded states, take a
    // write-back of the L2, by one wave after the barrier.  With a write-back
    // after and an invalidation before every item, and in every poll of the queue,
    // 32 workgroups kept emptying the L2 they share: uneven instances per launch 4
    // 4.51 -> 3.82 ms, 8 5.44 -> 4.50, 16 8.17 -> 6.44, 32 10.5 -> 9.9, 256 76.9 ->
    // 75.0.
    const bool fenced =
        phase == kPhShift || phase == kPhPaths || phase == kPhTopk || (phase == kPhRoll && P.n_dbg > 0);
    stores_done();
    __syncthreads();
    if (phase == kPhRoll) {
      const uint32_t lg = shape_roll_lg(shape);
      const uint32_t next = (tile << lg) + sub + 1u;
      if (sub + 1u < (1u << lg) && next < phase_tiles(P, kPhRoll, shape & ~make_shape(0, 0, 3, 0))) {
        ++sub;   // the same item's next tile (the barrier above ordered its LDS reuse)
        continue;
      }
      sub = 0;
    }

    if (tid == 0) {
      if (fenced) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      sh.publish = 0;
      const uint32_t nt = phase_tiles(P, phase, shape);
      const uint32_t done = atomicAdd(&ictl[inst].done, 1u) + 1u;
      if (done == nt) {
        atomicExch(&ictl[inst].done, 0u);
        uint32_t nph, nk;
        if (phase == kPhShift) {
          nph = kPhPaths; nk = ictl[inst].k_begin;
        } else if (phase == kPhUpd) {
          nph = kPhPaths; nk = k + 1u;
        } else {
          nph = phase + 1u; nk = k;
        }
        if (phase == kPhUpd && nk >= ictl[inst].k_end) {
          atomicAdd(&ctl->finished, 1u);
        } else {
          const uint32_t m = phase_tiles(P, nph, shape);
          sh.pub_pos = atomicAdd(&ctl->tail, m);
          sh.pub_count = m;
          sh.pub_phase = nph;
          sh.pub_k = nk;
          sh.publish = 1;
        }
      }
    }
    __syncthreads();
    if (sh.publish) {
      const uint32_t p0 = sh.pub_pos, m = sh.pub_count;
      if (p0 + m <= ctl->capacity) {
        for (uint32_t t = tid; t < m; t += kBatchThreads) {
          BatchItem it;
          it.inst = inst; it.phase = sh.pub_phase | (shape << kItemShapeShift); it.k = sh.pub_k; it.tile = t;
          store_item(&queue[p0 + t], it);
        }
        // wave 0 sets the ready flags once every wave's entries have reached memory
        stores_done();
        __syncthreads();
        if (tid < 64)
          for (uint32_t t = tid; t < m; t += 64)
            __hip_atomic_store(&ready[p0 + t], epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else if (tid == 0) {
        atomicOr(&ctl->error, 2u);   // queue overflow: items are never published, waiters time out
      }
    }
    __syncthreads();
  }
}

// Prepare one launch: per active instance record the replan index and shift,
// stage x0 and reset its tile counter; block 0 resets the queue and publishes
// one warm-start shift item per active instance in the given order.
__global__ __launch_bounds__(64) void k_batch_init(const PlanDesc* __restrict__ descs, InstCtl* __restrict__ ictl,
                                                   BatchCtl* ctl, BatchItem* __restrict__ queue,
                                                   uint32_t* __restrict__ ready, const int32_t* __restrict__ order,
                                                   int32_t n_active, uint32_t total, const float* __restrict__ x0_packed) {
  const int tid = threadIdx.x;
  const int slot = blockIdx.x;
  if (slot >= n_active) return;
  const int i = order[slot];
  const PlanDesc P = descs[i];
  const InstCtl ic = ictl[i];
  if (tid == 0) {
    P.ctrl[0] = ic.r;
    P.ctrl[1] = static_cast<uint32_t>(ic.k_begin == 0u ? ic.shift : 0);
    if (ic.k_begin == 0u) P.ctrl[2] = 0u;
    ictl[i].done = 0u;
  }
  if (x0_packed != nullptr && ic.x0_off >= 0)
    for (int e = tid; e < P.d; e += 64) P.x0[e] = x0_packed[ic.x0_off + e];
  if (tid == 0) {
    const uint32_t epoch = ctl->epoch + 1u;   // ctl is rewritten by the host-side reset below
    BatchItem it;
    it.inst = static_cast<uint32_t>(i);
    it.phase = kPhShift | (ic.shape << kItemShapeShift);
    it.k = ic.k_begin;
    it.tile = 0u;
    queue[slot] = it;
    ready[slot] = epoch;
  }
  (void)total;
}

__global__ void k_batch_reset(BatchCtl* ctl, int32_t n_active, uint32_t total) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    ctl->head = 0u;
    ctl->tail = static_cast<uint32_t>(n_active);
    ctl->total = total;
    ctl->finished = 0u;
    ctl->error = 0u;
    ctl->epoch = ctl->epoch + 1u;
  }
}

// Gather every active instance's action into one packed array and append the
// launch status (error flags, finished count).
__global__ __launch_bounds__(64) void k_batch_pack(const PlanDesc* __restrict__ descs, const InstCtl* __restrict__ ictl,
                                                   const BatchCtl* ctl, float* __restrict__ out, int32_t n_inst,
                                                   int32_t status_off) {
  const int i = blockIdx.x;
  if (i < n_inst) {
    const PlanDesc P = descs[i];
    const int off = ictl[i].act_off;
    for (int j = threadIdx.x; j < P.n; j += 64) out[off + j] = P.action[j];
  }
  if (i == 0 && threadIdx.x == 0) {
    uint32_t* st = reinterpret_cast<uint32_t*>(out + status_off);
    st[0] = ctl->error;
    st[1] = ctl->finished;
    st[2] = ctl->head;
  }
}

hipError_t launch_batch_prepare(const BatchLaunch& L, hipStream_t st) {
  k_batch_init<<<L.n_active, 64, 0, st>>>(L.descs, L.ictl, L.ctl, L.queue, L.ready, L.order, L.n_active, L.total,
                                          L.x0_packed);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_batch_reset<<<1, 64, 0, st>>>(L.ctl, L.n_active, L.total);
  return hipGetLastError();
}

hipError_t launch_batch_persistent(const BatchLaunch& L, int grid, hipStream_t st) {
  k_batch_persistent<<<grid, kBatchThreads, 0, st>>>(L.descs, L.ictl, L.ctl, L.queue, L.ready, L.wait_ticks);
  return hipGetLastError();
}

hipError_t launch_batch_pack(const BatchLaunch& L, float* out, int32_t n_inst, int32_t status_off, hipStream_t st) {
  k_batch_pack<<<n_inst, 64, 0, st>>>(L.descs, L.ictl, L.ctl, out, n_inst, status_off);
  return hipGetLastError();
}

int batch_max_blocks_per_cu() {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_batch_persistent, kBatchThreads, 0) != hipSuccess) return 1;
  return n > 0 ? n : 1;
}

}  // namespace mtp
