// Selection of few elites from few candidates by one wave: no barriers, so the
// workgroup's other waves work on meanwhile.
#pragma once

#include "mtp_device.hpp"

namespace mtp {

constexpr int kWaveKeys = 16;   // cost images per lane

// The E smallest of the n <= 64 kWaveKeys images that a wave holds (image i in
// o[i / 64] of lane i % 64, all-ones past n), ties to the lower i; put(slot, i,
// image) for each, slots in increasing i.  Returns how many (E, or n if less).
// The E-th smallest image is found bit by bit from the highest bit that differs,
// counting the images below the trial value with one ballot per 64 of them; it
// stops as soon as a trial value has exactly E below it.
template <class Put>
__device__ __forceinline__ int wave_smallest(const uint32_t (&o)[kWaveKeys], int lane, int n, int E, Put put) {
  const int rows = (n + 63) >> 6;   // n is the same for the whole wave
  uint32_t limit = 0xFFFFFFFFu;   // images below it are taken
  int ties = 0;                   // and this many of those equal to it
  if (n > E) {
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
    for (int g = 0; g < kWaveKeys; g += 4)
      if (g < rows) {
#pragma unroll
        for (int q = g; q < g + 4; ++q) {
          lo = min(lo, o[q]);
          hi = max(hi, o[q] == 0xFFFFFFFFu ? 0u : o[q]);
        }
      }
    lo = wave_min_u32(lo);
    hi = wave_max_u32(hi);
    const int bits = lo == hi ? 0 : 32 - __clz(static_cast<int>(lo ^ hi));
    uint32_t T = bits >= 32 ? 0u : (lo >> bits) << bits;
    int below = 0;   // images below T
    bool exact = false;
    for (int bit = bits - 1; bit >= 0; --bit) {
      const uint32_t trial = T | (1u << bit);
      uint32_t c = 0;
#pragma unroll
      for (int g = 0; g < kWaveKeys; g += 4)   // four independent counts at a time; all-ones images never count
        if (g < rows)
          c += (__popcll(__ballot(o[g] < trial)) + __popcll(__ballot(o[g + 1] < trial))) +
               (__popcll(__ballot(o[g + 2] < trial)) + __popcll(__ballot(o[g + 3] < trial)));
      if (c == static_cast<uint32_t>(E)) { limit = trial; exact = true; break; }
      if (c < static_cast<uint32_t>(E)) { T = trial; below = static_cast<int>(c); }
    }
    if (!exact) { limit = T; ties = E - below; }
  }
  int base = 0;
#pragma unroll
  for (int q = 0; q < kWaveKeys; ++q) {
    if (q < rows) {
      bool take = o[q] < limit;
      if (ties > 0) {
        const unsigned long long eq = __ballot(o[q] == limit);
        const int before = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(eq >> 32),
                                                     __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(eq), 0u));
        take = take || (o[q] == limit && before < ties);
        ties -= static_cast<int>(__popcll(eq));
      }
      const unsigned long long m = __ballot(take);
      const int slot = base + static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                                   __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u)));
      if (take) put(slot, lane + 64 * q, o[q]);
      base += static_cast<int>(__popcll(m));
    }
  }
  return base;
}

// The E smallest of n images (as wave_smallest) into list_o / list_b, from a
// bound on the E-th: the E-th smallest of the 64 lanes' smallest images.  At
// least E images are at or below it and seldom many more (16 of 288 uniform
// keys: about 20), and those are ordered by counting.  Returns how many are in
// the list, 0 if they would not fit.
__device__ __forceinline__ int wave_short_list(const uint32_t (&o)[kWaveKeys], int lane, int n, int E, uint32_t* mins,
                                               uint32_t* list_o, uint32_t* list_b) {
  uint32_t m = o[0];
#pragma unroll
  for (int q = 1; q < kWaveKeys; ++q) m = min(m, o[q]);
  // the lane's place among the minima, read back by all lanes alike (a lane
  // read per value would cost its latency sixty-four times), every read in
  // flight before the first use
  mins[lane] = m;
  int below = 0;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    uint4 x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = reinterpret_cast<const uint4*>(mins)[8 * h + j];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      below += ((x[j].x < m ? 1 : 0) + (x[j].y < m ? 1 : 0)) + ((x[j].z < m ? 1 : 0) + (x[j].w < m ? 1 : 0));
  }
  const uint32_t bound = wave_max_u32(below < E ? m : 0u);
  int total = 0;
#pragma unroll
  for (int q = 0; q < kWaveKeys; ++q) total += static_cast<int>(__popcll(__ballot(o[q] <= bound)));
  if (total > 64) return 0;
  int base = 0;
#pragma unroll
  for (int q = 0; q < kWaveKeys; ++q) {
    const bool take = o[q] <= bound;   // never an all-ones image
    const unsigned long long in = __ballot(take);
    if (in != 0ull) {
      const int slot = base + static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(in >> 32),
                                                   __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(in), 0u)));
      if (take) {
        list_o[slot] = o[q];
        list_b[slot] = static_cast<uint32_t>(lane + 64 * q);
      }
      base += static_cast<int>(__popcll(in));
    }
  }
  return total;
}

struct WaveSelectSmem {
  alignas(16) uint32_t mins[64], list_o[64];   // the lanes' smallest images; the short list's images
  uint32_t list_b[64];                         // and candidates, in candidate order
  unsigned long long sorted[64];
};

struct WaveElite {
  int idx;        // candidate of elite `lane` (lanes below E)
  float cost, weight, best;   // its cost and softmax weight (0 past the last elite); the best cost
};

// The E <= 64 elites of n images (as wave_smallest), in order, one per lane, with
// their softmax weights as topk_block forms them.  cost_of(idx, c) gives the cost
// of a candidate whose image says c.
template <class CostOf>
__device__ __forceinline__ WaveElite wave_elites(const uint32_t (&o)[kWaveKeys], int lane, int n, int E, float lam,
                                                 WaveSelectSmem& sm, CostOf cost_of) {
  int count = wave_short_list(o, lane, n, E, sm.mins, sm.list_o, sm.list_b);
  if (count == 0)
    count = wave_smallest(o, lane, n, E, [&](int slot, int b, uint32_t im) {
      sm.list_o[slot] = im;
      sm.list_b[slot] = static_cast<uint32_t>(b);
    });
  // order by counting (ties to the lower candidate, whose slot is lower)
  const uint32_t im = lane < count ? sm.list_o[lane] : 0xFFFFFFFFu, ib = sm.list_b[lane];
  sm.list_o[lane] = im;
  int rank = 0;
  for (int e0 = 0; e0 < count; e0 += 32) {   // at most twice
    uint4 x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = *reinterpret_cast<const uint4*>(&sm.list_o[e0 + 4 * j]);
    __builtin_amdgcn_sched_barrier(0);
    auto lower = [&](uint32_t v, int e) { return (v < im || (v == im && e < lane)) ? 1 : 0; };
#pragma unroll
    for (int j = 0; j < 8; ++j)
      rank += (lower(x[j].x, e0 + 4 * j) + lower(x[j].y, e0 + 4 * j + 1)) +
              (lower(x[j].z, e0 + 4 * j + 2) + lower(x[j].w, e0 + 4 * j + 3));
  }
  if (lane < count && rank < E) sm.sorted[rank] = (static_cast<unsigned long long>(im) << 32) | ib;
  // elites, their costs and softmax weights
  const unsigned long long mine = lane < E ? sm.sorted[lane] : 0ull;
  const int idx = static_cast<int>(static_cast<uint32_t>(mine));
  const float ce = cost_of(idx, order_cost(static_cast<uint32_t>(mine >> 32)));
  const float s0 = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(ce)));
  const bool uniform = !(lam < INFINITY) || !(s0 < INFINITY);
  const float raw = lane < E ? (uniform ? 1.0f : expf(-(ce - s0) / lam)) : 0.0f;
  const float inv = 1.0f / wave_sum64(raw);
  const float wv = raw * inv;
  return {idx, ce, wv, s0};
}

}  // namespace mtp
