// Candidate tiles of the batched launch.
//
// An item draws 256 candidates of every joint (or of one), so what the joints
// share is done once: the layer indices of the tensor paths are drawn once and
// packed, the graph columns of as many joints as fit in LDS come from whole
// Philox blocks (a block holds the values of four neighbouring joints), the
// spline tables are staged once, and the spline steps run two joints at a time.
// The values are those of cand_tile (the same arithmetic in the same order),
// which the single-plan kernels run on (tile, joint, horizon chunk) workgroups.
//
// What bounded the tile before was issue and waiting: the spline steps read four
// control values and a table row from LDS each, drew the indices again for every
// joint, and waited for earlier stores (see spline_steps).  256 uneven instances
// (43 GB of controls per replan): candidates 15.7 -> 10.3 ms per workgroup, replan
// 81.8 -> 77.0 ms; 32 instances 11.0 -> 10.5 ms.  With every unit drawing at once
// the stores bound it (4 TB/s).  Not used by the single plans' kernels: their
// launches draw one joint per workgroup beside rollouts, where this code's size
// cost more than it gave (seven links, 9216 candidates: replan 1.02 -> 1.04 ms).
#pragma once

#include "mtp_device.hpp"

namespace mtp {

constexpr int kGraphTile = 8192;    // graph values of the joints drawn at a time
constexpr int kBatchChunk = 256;    // horizon steps whose spline tables are staged at a time
constexpr int kJoints = 2;          // joints evaluated together

struct BatchCandSmem {
  float4 tb[kBatchChunk][kBasisStride / 4];      // spline weights of the staged steps
  int32_t ts[kBatchChunk];                       // their span / interval index
  float z[kGraphTile];                           // Z[l][w] of some joints
  float ctrl[kJoints][kMaxLayers][kCandThreads];    // per-thread control points
  float slope[kJoints][kMaxLayers][kCandThreads];   // per-thread Akima slopes (unit spacing)
};
static_assert(kGraphTile >= kMaxLayers * kMaxWidth, "at least one joint's column");

// A control of U, at agent scope (store_agent).
__device__ __forceinline__ void store_u(__attribute__((address_space(1))) float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The value lane `i` (uniform) of the wave holds.
__device__ __forceinline__ float lane_value(float v, int i) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), i));
}

// Tensor-path controls of joints [j, j + NJ), candidate b at the steps
// [t0, t1), at most 64: NP control values (load(jj, s, c) fetches those of span
// s) weighted by the step's table row (tb: the row of t0).  ZERO: the sum starts
// from zero, else from the first product.  Lane i of the wave holds the span of
// step t0 + i in `spans`; bit i of `change` is set where a span starts.
//
// A span holds for about T / (L - 3) steps, so its control values stay in
// registers: four steps inside one span are four broadcast reads of a table row,
// fetched while the four steps before are evaluated, and per joint NP
// multiply-adds, the clamp and the store each.  Nothing here loads from memory:
// stores share the loads' counter, and waiting for a load among them would wait
// until they have reached memory.
template <int NP, bool ZERO, int NJ, class Load>
__device__ __forceinline__ void spline_steps(const PlanDesc& P, const float4 (*tb)[kBasisStride / 4], int spans,
                                             uint64_t change, int j, int b, int t0, int t1, Load load) {
  constexpr int kG = 4, kQ = (NP + 3) / 4;
  typedef __attribute__((address_space(1))) char* OutPtr;
  const float lo = P.u_min;
  float hi = P.u_max;
  asm("" : "+v"(hi));   // one operand of the clamp has to be a vector register
  const size_t row = static_cast<size_t>(P.n) * P.ldU * sizeof(float);
  OutPtr out[NJ];
#pragma unroll
  for (int jj = 0; jj < NJ; ++jj) out[jj] = (OutPtr)(P.U + (static_cast<size_t>(t0) * P.n + j + jj) * P.ldU);
  float c[NJ][NP];
  struct Group { float4 w[kG][kQ]; };
  auto fetch = [&](int i0, Group& g) {
#pragma unroll
    for (int i = 0; i < kG; ++i)
#pragma unroll
      for (int q = 0; q < kQ; ++q) g.w[i][q] = tb[i0 + i][q];
  };
  auto value = [&](const float4 (&w)[kQ], int jj) {
    const float* wf = reinterpret_cast<const float*>(&w[0]);
    float v = ZERO ? fmaf(wf[0], c[jj][0], 0.0f) : wf[0] * c[jj][0];
#pragma unroll
    for (int q = 1; q < NP; ++q) v = fmaf(wf[q], c[jj][q], v);
    return __builtin_amdgcn_fmed3f(v, lo, hi);
  };
  // the control values are waited for here: left pending, every later use would
  // wait for the table rows in flight as well
  auto reload = [&](int i) {
    const int s = __builtin_amdgcn_readlane(spans, i);
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) load(jj, s, c[jj]);
    __builtin_amdgcn_s_waitcnt(0xC07F);   // LDS
  };
  const int n = t1 - t0;
  int i0 = 0;
  reload(0);
  change &= ~uint64_t{1};
  if (n >= kG && 64 * row + 4u * static_cast<size_t>(P.B) < (size_t(1) << 32)) {
    // 32-bit lane offsets to the joints' scalar bases
    uint32_t off[kG];
#pragma unroll
    for (int i = 0; i < kG; ++i) off[i] = static_cast<uint32_t>(b) * 4u + static_cast<uint32_t>(i * row);
    auto eval = [&](const Group& g) {
      float v[NJ][kG];
      const uint32_t starts = static_cast<uint32_t>(change >> i0) & 0xFu;
      if (starts == 0u) {
#pragma unroll
        for (int i = 0; i < kG; ++i)
#pragma unroll
          for (int jj = 0; jj < NJ; ++jj) v[jj][i] = value(g.w[i], jj);
      } else {
#pragma unroll
        for (int i = 0; i < kG; ++i) {
          if (starts & (1u << i)) reload(i0 + i);
#pragma unroll
          for (int jj = 0; jj < NJ; ++jj) v[jj][i] = value(g.w[i], jj);
        }
      }
#pragma unroll
      for (int i = 0; i < kG; ++i) {
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj)
          store_u((__attribute__((address_space(1))) float*)(out[jj] + off[i]), v[jj][i]);
        off[i] += static_cast<uint32_t>(kG * row);
      }
      i0 += kG;
    };
    const int last = n - kG;
    Group ga, gb;
    fetch(0, ga);
    for (;;) {
      fetch(min(i0 + kG, last), gb);
      eval(ga);
      if (i0 > last) break;
      fetch(min(i0 + kG, last), ga);
      eval(gb);
      if (i0 > last) break;
    }
  }
  for (; i0 < n; ++i0) {
    if ((change >> i0) & 1u) reload(i0);
    float4 w[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) w[q] = tb[i0][q];
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj)
      store_u((__attribute__((address_space(1))) float*)(out[jj] + i0 * row) + b, value(w, jj));
  }
}

// Tensor-path controls of joints [j, j + NJ) over steps [tc, te), staged in sm:
// control points from the packed layer indices, slopes, spline.
template <int NJ>
__device__ __forceinline__ void tensor_joints(const PlanDesc& P, BatchCandSmem& sm, const float* z,
                                              const uint32_t (&idx)[kMaxLayers / 4], bool is_tensor, int j, int b, int tc,
                                              int te) {
  const int tid = threadIdx.x, lane = tid & 63;
  if (is_tensor) {
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
      const float* zj = z + jj * P.L * P.W;
#pragma unroll
      for (int g = 0; g < kMaxLayers / 4; ++g) {
        if (4 * g + 3 < P.L) {
          float v[4];
#pragma unroll
          for (int c = 0; c < 4; ++c) v[c] = zj[(4 * g + c) * P.W + ((idx[g] >> (8 * c)) & 0xFFu)];
#pragma unroll
          for (int c = 0; c < 4; ++c) sm.ctrl[jj][4 * g + c][tid] = v[c];
        } else {
#pragma unroll
          for (int c = 0; c < 3; ++c)
            if (4 * g + c < P.L) sm.ctrl[jj][4 * g + c][tid] = zj[(4 * g + c) * P.W + ((idx[g] >> (8 * c)) & 0xFFu)];
        }
      }
      if (P.interp == kAkima) {
        CandView v;
        v.ctrl = &sm.ctrl[jj][0][0];
        v.slope = &sm.slope[jj][0][0];
        akima_slopes_thread(P.L, tid, v);
      }
    }
  }
  auto window = [&](int jj, int s, auto& c) {
#pragma unroll
    for (int q = 0; q < static_cast<int>(sizeof(c) / sizeof(float)); ++q) c[q] = sm.ctrl[jj][s + q][tid];
  };
  for (int t0 = tc; t0 < te; t0 += 64) {
    const int t1 = min(t0 + 64, te);
    const int at = min(t0 + lane, te - 1) - tc;
    const int spans = sm.ts[at];
    const uint64_t change = __ballot(spans != sm.ts[max(at - 1, 0)]);
    const auto tb = &sm.tb[t0 - tc];
    if (!is_tensor) continue;
    if (P.interp == kAkima) {
      spline_steps<4, false, NJ>(P, tb, spans, change, j, b, t0, t1, [&](int jj, int s, float (&c)[4]) {
        c[0] = sm.ctrl[jj][s][tid];
        c[1] = sm.slope[jj][s][tid];
        c[2] = sm.ctrl[jj][s + 1][tid];
        c[3] = sm.slope[jj][s + 1][tid];
      });
      continue;
    }
    switch (P.interp == kLinear ? 1 : P.p) {
      case 1: spline_steps<2, true, NJ>(P, tb, spans, change, j, b, t0, t1, window); break;
      case 2: spline_steps<3, true, NJ>(P, tb, spans, change, j, b, t0, t1, window); break;
      case 3: spline_steps<4, false, NJ>(P, tb, spans, change, j, b, t0, t1, window); break;
      case 4: spline_steps<5, true, NJ>(P, tb, spans, change, j, b, t0, t1, window); break;
      default: spline_steps<6, true, NJ>(P, tb, spans, change, j, b, t0, t1, window); break;
    }
  }
}

// Candidates [b0, b0 + kCandThreads) of joints [j0, j1) over the horizon.  The
// tile holding the first tensor path stores the graph columns to Z, and tiles of
// joint 0 store the path indices I (without replacement the path tiles have
// written both).  Every thread of the workgroup must call this (it synchronises
// the workgroup).
__device__ __forceinline__ void batch_cand_tile(const PlanDesc& P, uint32_t r, int k, int j0, int j1, int b0,
                                                BatchCandSmem& sm) {
  const auto Ug = gptr(P.U);
  const auto Zg = gptr(P.Z);
  const auto Ig = gptr(P.I);
  const int tid = threadIdx.x, lane = tid & 63, wave_b = b0 + (tid & ~63);
  const int b = b0 + tid;
  const int G1 = P.G - 1;                       // local samples [0, G1)
  const int tens_lo = G1, tens_hi = G1 + P.P;   // tensor paths [G1, G1+P)
  const bool tile_has_tensor = b0 < tens_hi && b0 + kCandThreads > tens_lo;
  const bool wave_has_tensor = wave_b < tens_hi && wave_b + 64 > tens_lo;
  const float lo = P.u_min, hi = P.u_max;
  const size_t ld = static_cast<size_t>(P.ldU);
  const bool is_local = b < G1;
  const bool is_tensor = b >= tens_lo && b < tens_hi;
  const int LW = P.L * P.W, Tq = (P.T + 3) >> 2;
  const int group = min(j1 - j0, kGraphTile / LW);   // joints whose columns are drawn at a time

  uint32_t idx[kMaxLayers / 4];   // layer l's index: byte l mod 4 of word l / 4
  if (is_tensor) {
    const int pp = b - G1;
    const bool i_writer = !P.wor && j0 == 0;
#pragma unroll
    for (int g = 0; g < kMaxLayers / 4; ++g) {
      idx[g] = 0u;
      if (4 * g >= P.L) continue;
      Words4 q;
      if (!P.wor)
        q = philox(static_cast<uint32_t>(g), static_cast<uint32_t>(pp), r, stream_c3(kTagI, k), P.key0, P.key1);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int l = 4 * g + c;
        if (l < P.L) {
          const size_t at = static_cast<size_t>(l) * P.P + pp;
          const uint32_t wi = P.wor ? static_cast<uint32_t>(Ig[at]) : __umulhi(q.w[c], static_cast<uint32_t>(P.W));
          idx[g] |= wi << (8 * c);
          if (i_writer) store_agent(&P.I[at], static_cast<uint8_t>(wi));
        }
      }
    }
  }

  for (int tc = 0; tc < P.T; tc += kBatchChunk) {
    const int te = min(tc + kBatchChunk, P.T);
    for (int jg = j0; jg < j1; jg += group) {
      const int je = min(jg + group, j1);
      if (tile_has_tensor) {
        // tables and graph columns, then one barrier
        if (tc != 0 || jg != j0) __syncthreads();   // the previous ones are read
        if (jg == j0) {
          for (int i = tid; i < te - tc; i += kCandThreads) sm.ts[i] = gptr(P.span)[tc + i];
          for (int i = tid; i < (te - tc) * kBasisStride; i += kCandThreads)
            reinterpret_cast<float*>(&sm.tb[0][0])[i] = gptr(P.basis)[tc * kBasisStride + i];
        }
        if (tc != 0 && group == j1 - j0) {
          // every column is there
        } else if (P.wor) {
          for (int e = tid; e < LW; e += kCandThreads)
            for (int j = jg; j < je; ++j) sm.z[(j - jg) * LW + e] = Zg[static_cast<size_t>(e) * P.n + j];
        } else {
          const bool z_writer = b0 <= tens_lo && tc == 0;
          const float span = hi - lo;
          for (int e = tid; e < LW; e += kCandThreads) {
            const int l = e / P.W, w = e - l * P.W;
            const int first = w * P.n + jg, last = w * P.n + je - 1;
            for (int blk = first >> 2; blk <= (last >> 2); ++blk) {
              const Words4 q = philox(static_cast<uint32_t>(blk), static_cast<uint32_t>(l), r, stream_c3(kTagZ, k),
                                      P.key0, P.key1);
#pragma unroll
              for (int c = 0; c < 4; ++c) {
                const int i = 4 * blk + c;
                if (i >= first && i <= last) {
                  const float z = fmaf(span, u01(q.w[c]), lo);
                  sm.z[(i - first) * LW + e] = z;
                  if (z_writer) store_agent(&P.Z[static_cast<size_t>(l) * P.W * P.n + i], z);
                }
              }
            }
          }
        }
        __syncthreads();
      }
      if (wave_has_tensor) {
        int j = jg;
        for (; j + kJoints <= je; j += kJoints)
          tensor_joints<kJoints>(P, sm, sm.z + (j - jg) * LW, idx, is_tensor, j, b, tc, te);
        for (; j < je; ++j) tensor_joints<1>(P, sm, sm.z + (j - jg) * LW, idx, is_tensor, j, b, tc, te);
      }
      if (wave_b < G1) {
        // Local sample g = b: u = clip(mu + sigma * eps), four steps per Philox
        // block.  The wave loads a joint's moments of the whole chunk at once, one
        // step per lane and register (a load per block would wait for the previous
        // block's stores).
        constexpr int kRegs = kBatchChunk / 64;
        const size_t row = static_cast<size_t>(P.n) * ld;
        float hv = hi;
        asm("" : "+v"(hv));   // one operand of the clamp has to be a vector register
        for (int j = jg; j < je; ++j) {
          float mu[kRegs], sg[kRegs];
#pragma unroll
          for (int i = 0; i < kRegs; ++i) {
            const int o = min(tc + 64 * i + lane, te - 1) * P.n + j;
            mu[i] = gptr(P.mu)[o];
            sg[i] = gptr(P.sigma)[o];
          }
          for (int t0 = tc; t0 < te; t0 += 64) {
            const int t1 = min(t0 + 64, te);
            if (is_local) {
              auto out = Ug + (static_cast<size_t>(t0) * P.n + j) * ld + b;
              // normals of the four steps from t4 on
              auto normals = [&](int t4, float (&z)[4]) {
                const Words4 q = philox(static_cast<uint32_t>(j * Tq + (t4 >> 2)), static_cast<uint32_t>(b), r,
                                        stream_c3(kTagEps, k), P.key0, P.key1);
                box_muller(q.w[0], q.w[1], z[0], z[1]);
                box_muller(q.w[2], q.w[3], z[2], z[3]);
              };
              auto put = [&](int t, float z) {
                const float v = fmaf(lane_value(sg[0], t - t0), z, lane_value(mu[0], t - t0));
                store_u(out, __builtin_amdgcn_fmed3f(v, lo, hv));
                out += row;
              };
              int t4 = t0;
              for (; t4 + 8 <= t1; t4 += 8) {   // two blocks' chains side by side
                float z[2][4];
                normals(t4, z[0]);
                normals(t4 + 4, z[1]);
#pragma unroll
                for (int c = 0; c < 8; ++c) put(t4 + c, z[c >> 2][c & 3]);
              }
              for (; t4 < t1; t4 += 4) {
                float z[4];
                normals(t4, z);
#pragma unroll
                for (int c = 0; c < 4; ++c)
                  if (t4 + c < t1) put(t4 + c, z[c]);
              }
            }
#pragma unroll
            for (int i = 0; i + 1 < kRegs; ++i) { mu[i] = mu[i + 1]; sg[i] = sg[i + 1]; }   // the next 64 steps
          }
        }
      }
      if (tens_hi >= b0 && tens_hi < b0 + kCandThreads) {
        // nominal mean, one step per thread
        for (int j = jg; j < je; ++j)
          for (int t = tc + tid; t < te; t += kCandThreads)
            store_u(&Ug[(static_cast<size_t>(t) * P.n + j) * ld + tens_hi],
                    clampf(gptr(P.mu)[t * P.n + j], lo, hi));
      }
    }
  }
}

}  // namespace mtp
