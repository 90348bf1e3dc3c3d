// A whole point-mass replan in two kernels, for plans with few local samples.
//
// The staged replan of a point mass runs three launches per CEM iteration whose
// work is a few microseconds each.  The tensor paths of every iteration, and so
// their costs, depend on nothing but the seed and the start state: k_pm_tensor
// rolls out all iterations' tensor paths at once, over the whole chip.  What is
// left of an iteration, the local samples' rollout, the selection over all
// costs and the refit, is small enough for one workgroup: k_pm_iterate runs all
// iterations with workgroup barriers between the stages instead of launches.
// Every operation and its order are those of the staged kernels, so the results
// are the same bits.  Long replans run in chunks of kPmChunk iterations, so that
// the kept costs and a launch's time stay bounded.
//
// What bounds an iteration is the latency of its chain (about ten dependent
// phases on one compute unit); the normals and the graph of the next iteration
// are drawn by the waves that wait while one wave selects.  Per iteration of 288
// candidates x 50 steps, of about 9 us: controls 1.1, states 0.9, cost terms 1.9
// (the one phase bound by issue: 20 obstacle tests for each of 1600 points on
// one compute unit), their sums 0.6, selection 2.7, refit 1.9.  Replans before
// -> now: 288 x 50 x 10 iterations 0.187 -> 0.096 ms; 256 x 20 x 10
// 0.171 -> 0.075 ms.
#include <algorithm>

#include "kernels.hpp"
#include "pm_tile.hpp"
#include "wave_select.hpp"

namespace mtp {

namespace {

constexpr int kTensorTile = 16;       // tensor paths per workgroup of k_pm_tensor
constexpr int kTensorThreads = 256;
constexpr int kIterThreads = 1024;

// The whole graph of iteration k in LDS, [layer][waypoint][2] (Def. 1), drawn by
// `stride` threads of which this is number `first`.
__device__ __forceinline__ void draw_graph(const PlanDesc& P, uint32_t r, int k, float* z, int first, int stride) {
  const int Wn = 2 * P.W, nb = (Wn + 3) >> 2;
  const float lo = P.u_min, span = P.u_max - P.u_min;
  for (int e = first; e < P.L * nb; e += stride) {
    const int l = e / nb, blk = e - l * nb;
    const Words4 q = philox(static_cast<uint32_t>(blk), static_cast<uint32_t>(l), r, stream_c3(kTagZ, k), P.key0, P.key1);
#pragma unroll
    for (int w = 0; w < 4; ++w)
      if (4 * blk + w < Wn) z[l * Wn + 4 * blk + w] = fmaf(span, u01(q.w[w]), lo);
  }
}

// Layer indices of tensor path p (Alg. 1): put(l, w) for every layer of [l4, l4 + 4).
template <class Put>
__device__ __forceinline__ void draw_indices(const PlanDesc& P, uint32_t r, int k, int p, int l4, Put put) {
  const Words4 q = philox(static_cast<uint32_t>(l4), static_cast<uint32_t>(p), r, stream_c3(kTagI, k), P.key0, P.key1);
#pragma unroll
  for (int c = 0; c < 4; ++c)
    if (4 * l4 + c < P.L) put(4 * l4 + c, __umulhi(q.w[c], static_cast<uint32_t>(P.W)));
}

// Akima slope at layer i of the control points ct(l) (the rules of akima_slopes_thread).
template <class Ct>
__device__ __forceinline__ float akima_slope(int L, int i, Ct ct) {
  if (i == 0) return ct(1) - ct(0);
  if (i == L - 1) return ct(L - 1) - ct(L - 2);
  if (i == 1) return 0.5f * (ct(2) - ct(0));
  if (i == L - 2) return 0.5f * (ct(L - 1) - ct(L - 3));
  const float m2 = ct(i - 1) - ct(i - 2);
  const float m1 = ct(i) - ct(i - 1);
  const float m0 = ct(i + 1) - ct(i);
  const float mp = ct(i + 2) - ct(i + 1);
  const float wa = fabsf(mp - m0);
  const float wb = fabsf(m1 - m2);
  const float den = wa + wb;
  return (den == 0.0f) ? 0.5f * (m1 + m0) : (wa * m1 + wb * m0) / den;
}

// Control of a tensor path with control points ct(l) and Akima slopes sl(l) at
// the step whose table row is bw and whose first layer (interval) is s0, as
// cand_tile evaluates it.
template <class Ct, class Sl>
__device__ __forceinline__ float tensor_control(const PlanDesc& P, const float* bw, int s0, Ct ct, Sl sl) {
  float v;
  if (P.interp == kAkima) {
    v = bw[0] * ct(s0);
    v = fmaf(bw[1], sl(s0), v);
    v = fmaf(bw[2], ct(s0 + 1), v);
    v = fmaf(bw[3], sl(s0 + 1), v);
  } else if (P.interp == kBspline && P.p == 3) {
    v = bw[0] * ct(s0);
    v = fmaf(bw[1], ct(s0 + 1), v);
    v = fmaf(bw[2], ct(s0 + 2), v);
    v = fmaf(bw[3], ct(s0 + 3), v);
  } else {
    const int np1 = P.interp == kLinear ? 2 : P.p + 1;
    v = 0.0f;
    for (int q = 0; q < np1; ++q) v = fmaf(bw[q], ct(s0 + q), v);
  }
  return clampf(v, P.u_min, P.u_max);
}

// What a launch runs: all iterations, or a range (kernels of its own: with the
// bounds as values whole replans take 1 to 2 % longer).
struct WholeReplan {
  __device__ int begin(const PlanDesc&) const { return 0; }
  __device__ int end(const PlanDesc& P) const { return P.K; }
};
struct IterRange {
  int k0, k1;
  __device__ int begin(const PlanDesc&) const { return k0; }
  __device__ int end(const PlanDesc&) const { return k1; }
};

// ------------------------------------------------------------------ tensor paths of all iterations
struct TensorSmem {
  PmTile<kTensorTile> tile;
  float z[kPmGraph];
  float4 obs[kMaxObstacles];
  float tb[kTileSteps * kBasisStride];
  int32_t ts[kTileSteps];
  float ctp[kMaxLayers][2][kTensorTile], slp[kMaxLayers][2][kTensorTile];   // control points, Akima slopes
};

// Workgroup (tile, i): the costs of tensor paths 16 tile .. of the range's iteration i;
// the last iteration's also leave their controls, indices and graph where the
// staged kernels do.  Workgroup (0, 0) records the replan (as k_set_ctrl).
template <class Range>
__global__ __launch_bounds__(kTensorThreads) void k_pm_tensor(PlanDesc P, uint32_t r, int shift,
                                                              const float* __restrict__ x0_src, Range range) {
  __shared__ TensorSmem sm;
  const int tid = threadIdx.x;
  const int k = range.begin(P) + static_cast<int>(blockIdx.y);
  const bool keep = k == P.K - 1;
  if (blockIdx.x == 0 && k == 0) {
    if (tid < 4) P.x0[tid] = x0_src[tid];
    if (tid == 0) {
      P.ctrl[0] = r;
      P.ctrl[1] = static_cast<uint32_t>(shift);
      P.ctrl[2] = 0u;
      P.ctrl[4] = 0u;
      P.ctrl[5] = 0u;
    }
  }
  const int p0 = static_cast<int>(blockIdx.x) * kTensorTile;
  if (p0 >= P.P) return;   // no tensor paths: the one workgroup per iteration that is launched anyway
  const int n_pad = load_obstacles(P, sm.obs);
  draw_graph(P, r, k, sm.z, tid, kTensorThreads);
  __syncthreads();
  for (int e = tid; e < kTensorTile * ((P.L + 3) >> 2); e += kTensorThreads) {
    const int c = e % kTensorTile, p = p0 + c;
    draw_indices(P, r, k, min(p, P.P - 1), e / kTensorTile, [&](int l, uint32_t w) {
      sm.ctp[l][0][c] = sm.z[(l * P.W + static_cast<int>(w)) * 2];
      sm.ctp[l][1][c] = sm.z[(l * P.W + static_cast<int>(w)) * 2 + 1];
      if (keep && p < P.P) P.I[static_cast<size_t>(l) * P.P + p] = static_cast<uint8_t>(w);
    });
  }
  __syncthreads();
  if (keep && blockIdx.x == 0)
    for (int e = tid; e < P.L * P.W * 2; e += kTensorThreads) P.Z[e] = sm.z[e];
  if (P.interp == kAkima) {
    for (int e = tid; e < P.L * 2 * kTensorTile; e += kTensorThreads) {
      const int c = e % kTensorTile, j = (e / kTensorTile) & 1, l = e / (2 * kTensorTile);
      sm.slp[l][j][c] = akima_slope(P.L, l, [&](int i) { return sm.ctp[i][j][c]; });
    }
    __syncthreads();
  }
  PlanDesc Q = P;
  Q.x0 = const_cast<float*>(x0_src);   // P.x0 is being written by this launch
  const float cost = pm_tile_cost<kTensorTile, kTensorThreads>(Q, sm.tile, sm.obs, n_pad, [&](int t0, int steps) {
    if (t0 > 0) __syncthreads();
    for (int i = tid; i < steps; i += kTensorThreads) sm.ts[i] = P.span[t0 + i];
    for (int i = tid; i < steps * kBasisStride; i += kTensorThreads) sm.tb[i] = P.basis[t0 * kBasisStride + i];
    __syncthreads();
    const int c = tid % kTensorTile, j = (tid / kTensorTile) & 1;
    auto ct = [&](int l) { return sm.ctp[l][j][c]; };
    auto sl = [&](int l) { return sm.slp[l][j][c]; };
    for (int i = tid / (2 * kTensorTile); i < steps; i += kTensorThreads / (2 * kTensorTile)) {
      const float v = tensor_control(P, sm.tb + i * kBasisStride, sm.ts[i], ct, sl);
      sm.tile.u[i][j][c] = v;
      if (keep && p0 + c < P.P)
        P.U[static_cast<size_t>((t0 + i) * 2 + j) * P.ldU + (P.G - 1 + p0 + c)] = v;
    }
  }, [](int, int, int, float, float) {});
  if (tid < kTensorTile && p0 + tid < P.P) {
    P.pm_cost[static_cast<size_t>(blockIdx.y) * P.P + p0 + tid] = cost;
    if (keep) P.cost[P.G - 1 + p0 + tid] = cost;
  }
}

// Sum of 64 values in wave_sum64's order (a balanced tree over the lanes), the
// quad's lane s holding values 16 s .. 16 s + 15.
__device__ __forceinline__ float quad_tree64(float (&a)[16]) {
#pragma unroll
  for (int h = 1; h < 16; h <<= 1)
#pragma unroll
    for (int i = 0; i < 16; i += 2 * h) a[i] += a[i + h];
  return quad_sum(a[0]);
}

// ------------------------------------------------------------------ the iterations
template <int C>
struct IterSmem {
  union {
    PmTile<C> tile;                       // local samples' rollout
    float vals[kPmValues];                // elite controls [elite][output]
  };
  float4 obs[kMaxObstacles];
  float z[2][kPmGraph];                   // graph of this and of the next iteration
  float normals[2][kPmNormals];           // local samples' normals [2 t + j][g], this and the next iteration's
  float tb[kPmSteps * kBasisStride];
  int32_t ts[kPmSteps];
  float mu[2][kPmSteps * 2], sg[2][kPmSteps * 2];   // current moments and the refit's
  // cost images of the candidates, all-ones past the last, of this and the next iteration
  uint32_t image[2][64 * kWaveKeys];
  WaveSelectSmem sel;
  int32_t eidx[kPmElites];
  float w[kPmElites];
  float ctp[kMaxLayers][2][kPmElites], slp[kMaxLayers][2][kPmElites];   // the elites' control points, Akima slopes
};

// The iterations of the range, from the moments that the previous ones left.
template <int C, class Range>
__global__ __launch_bounds__(kIterThreads) void k_pm_iterate(PlanDesc P, Range range) {
  const int k0 = range.begin(P), k1 = range.end(P);
  __shared__ IterSmem<C> sm;
  int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t r = P.ctrl[0];
  const int Tn = P.T * 2, G1 = P.G - 1, Tq = (P.T + 3) >> 2;
  const float lo = P.u_min, hi = P.u_max;
  // normals of iteration k's local samples, four steps per Philox block, by
  // `stride` threads of which this is number `first`
  auto draw_normals = [&](int k, float* out, int first, int stride) {
    for (int a = first; a < 2 * Tq * G1; a += stride) {
      const int g = a % G1, rest = a / G1, j = rest & 1, tq = rest >> 1;
      float z[4];
      local_normals4(P, tq, j, g, k, r, z);
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (4 * tq + c < P.T) out[((4 * tq + c) * 2 + j) * G1 + g] = z[c];
    }
  };
  const int n_pad = load_obstacles(P, sm.obs);
  for (int i = tid; i < P.T; i += kIterThreads) sm.ts[i] = P.span[i];
  for (int i = tid; i < P.T * kBasisStride; i += kIterThreads) sm.tb[i] = P.basis[i];
  {
    // the warm start, shifted (as shift_block), or the moments as they are
    const int s = k0 == 0 ? min(static_cast<int>(P.ctrl[1]), P.T) : 0;
    for (int e = tid; e < Tn; e += kIterThreads) {
      const int t = e >> 1, j = e & 1;
      sm.mu[0][e] = P.mu[s == 0 ? e : (t < P.T - s ? e + 2 * s : (P.T - 1) * 2 + j)];
      sm.sg[0][e] = t < P.T - s ? P.sigma[e + 2 * s] : P.sigma_init;
    }
  }
  // tensor paths' cost images of iteration k
  auto take_tensor = [&](int k, uint32_t* image, int first, int stride) {
    for (int p = first; p < P.P; p += stride) image[G1 + p] = cost_order(P.pm_cost[static_cast<size_t>(k - k0) * P.P + p]);
  };
  for (int b = P.B + tid; b < 64 * kWaveKeys; b += kIterThreads) sm.image[0][b] = sm.image[1][b] = 0xFFFFFFFFu;
  take_tensor(k0, sm.image[0], tid, kIterThreads);
  draw_graph(P, r, k0, sm.z[0], tid, kIterThreads);
  draw_normals(k0, sm.normals[0], tid, kIterThreads);
  __syncthreads();

  for (int k = k0; k < k1; ++k) {
    // addresses and masks are made again in every iteration: kept across them
    // they do not fit the registers, and each use would wait for its reload
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const int cur = (k - k0) & 1;   // buffers of this iteration; the others are the next one's
    const bool stop = k == k1 - 1, last = stop && k1 == P.K;   // the launch's last, the replan's
    const float* mu = sm.mu[cur];
    const float* sg = sm.sg[cur];
    const float* nz = sm.normals[cur];

    // local samples and the nominal: controls, rollout
    const float cost_own = pm_tile_cost<C, kIterThreads>(
        P, sm.tile, sm.obs, n_pad,
        [&](int t0, int steps) {
          for (int a = tid; a < 2 * C * steps; a += kIterThreads) {
            const int c = a % C, o = 2 * t0 + a / C;
            const float m = mu[o], s = sg[o], z = nz[o * G1 + min(c, max(G1 - 1, 0))];
            // past the nominal: idle lanes take the nominal's controls
            const float v = clampf(c < G1 ? fmaf(s, z, m) : m, lo, hi);
            (&sm.tile.u[0][0][0])[a] = v;
            if (last && c < P.G) P.U[static_cast<size_t>(o) * P.ldU + (c < G1 ? c : P.B - 1)] = v;
          }
        },
        [](int, int, int, float, float) {});
    if (tid < C && tid < P.G) {
      sm.image[cur][tid < G1 ? tid : P.B - 1] = cost_order(cost_own);
      if (last) P.cost[tid < G1 ? tid : P.B - 1] = cost_own;
    }
    __syncthreads();

    if (wave == 0) {
      // selection: one wave, no barriers, ahead of the other waves' drawing
      __builtin_amdgcn_s_setprio(3);
      uint32_t o[kWaveKeys];
#pragma unroll
      for (int q = 0; q < kWaveKeys; ++q) o[q] = sm.image[cur][lane + 64 * q];
      // a cost is never NaN or -0 (finite_or_inf of a sum that starts at +0), so
      // its image gives it back
      const WaveElite el = wave_elites(o, lane, P.B, P.E, P.lam, sm.sel, [](int, float c) { return c; });
      const int idx = el.idx;
      const float ce = el.cost, s0 = el.best, wv = el.weight;
      sm.w[lane] = wv;   // 0 past the last elite
      if (lane < P.E) {
        sm.eidx[lane] = idx;
        if (last) {
          P.eidx[lane] = idx;
          P.ecost[lane] = ce;
          P.w[lane] = wv;
        }
      }
      if (lane == 0 && !(s0 < INFINITY)) atomicOr(&P.ctrl[2], 1u);
      __builtin_amdgcn_s_setprio(0);
    } else if (!stop && (wave & 3) != 0) {
      // the waves of the other three SIMDs prepare the next iteration meanwhile
      const int first = (wave - 1 - (wave >> 2)) * 64 + lane;
      constexpr int kHelpers = kIterThreads / 4 * 3;
      take_tensor(k + 1, sm.image[cur ^ 1], first, kHelpers);
      draw_graph(P, r, k + 1, sm.z[cur ^ 1], first, kHelpers);
      draw_normals(k + 1, sm.normals[cur ^ 1], first, kHelpers);
    }
    __syncthreads();

    // the tensor elites' control points
    const float* zt = sm.z[cur];
    for (int a = tid; a < P.E * ((P.L + 3) >> 2); a += kIterThreads) {
      const int e = a % P.E, b = sm.eidx[e];
      if (b >= G1 && b < G1 + P.P)
        draw_indices(P, r, k, b - G1, a / P.E, [&](int l, uint32_t w) {
          sm.ctp[l][0][e] = zt[(l * P.W + static_cast<int>(w)) * 2];
          sm.ctp[l][1][e] = zt[(l * P.W + static_cast<int>(w)) * 2 + 1];
        });
    }
    __syncthreads();
    if (P.interp == kAkima) {
      for (int a = tid; a < P.L * 2 * P.E; a += kIterThreads) {
        const int e = a % P.E, j = (a / P.E) & 1, l = a / (2 * P.E), b = sm.eidx[e];
        if (b >= G1 && b < G1 + P.P) sm.slp[l][j][e] = akima_slope(P.L, l, [&](int i) { return sm.ctp[i][j][e]; });
      }
      __syncthreads();
    }
    // refit: the elites' controls into LDS, then each output's sums on a quad of lanes
    // (the steps fastest, so that a wave's lanes mostly take the same kind of elite)
    for (int a = tid; a < P.E * Tn; a += kIterThreads) {
      const int o = a % Tn, e = a / Tn, b = sm.eidx[e], t = o >> 1, j = o & 1;
      float v;
      if (b >= G1 && b < G1 + P.P) {
        v = tensor_control(P, sm.tb + t * kBasisStride, sm.ts[t], [&](int l) { return sm.ctp[l][j][e]; },
                           [&](int l) { return sm.slp[l][j][e]; });
      } else {
        const float m = mu[o], s = sg[o], z = nz[o * G1 + min(b, max(G1 - 1, 0))];
        v = clampf(b < G1 ? fmaf(s, z, m) : m, lo, hi);
      }
      sm.vals[e * Tn + o] = v;
    }
    __syncthreads();
    // the sums of update_output: lane e of its wave holds elite e, summed by
    // wave_sum64; here quad lane s holds elites 16 s ..
    for (int a = tid; a < 4 * ((Tn + 15) & ~15); a += kIterThreads) {
      const int o = min(a >> 2, Tn - 1), s = a & 3;
      float val[16], wt[16], acc[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int e = 16 * s + i;
        val[i] = sm.vals[min(e, P.E - 1) * Tn + o];
        wt[i] = sm.w[e];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[i] = fmaf(wt[i], val[i], 0.0f);   // a product not fused into the tree
      const float m = quad_tree64(acc);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float dv = val[i] - m;
        acc[i] = fmaf(wt[i], dv * dv, 0.0f);
      }
      const float var = quad_tree64(acc);
      const float sd = fmaxf(sqrtf(var), P.sigma_min);
      const float mn = fmaf(P.alpha, mu[o] - m, m);
      const float sn = fmaf(P.alpha, sg[o] - sd, sd);
      if (s == 0 && (a >> 2) < Tn) {
        sm.mu[cur ^ 1][o] = mn;
        sm.sg[cur ^ 1][o] = sn;
        if (stop) {
          P.mu[o] = mn;
          P.sigma[o] = sn;
          if (o < 2) P.action[o] = val[0];   // the last chunk's is the replan's
        }
      }
    }
    __syncthreads();
  }
}

template <class Range>
hipError_t launch_range(const PlanDesc& P, uint32_t r, int shift, const float* x0_src, int iters, Range range,
                        hipStream_t st) {
  const dim3 grid(std::max(1, (P.P + kTensorTile - 1) / kTensorTile), iters);
  k_pm_tensor<<<grid, kTensorThreads, 0, st>>>(P, r, shift, x0_src, range);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // the tile's width follows the local candidates: idle lanes cost as much as others
  if (P.G <= 4) k_pm_iterate<4><<<1, kIterThreads, 0, st>>>(P, range);
  else if (P.G <= 16) k_pm_iterate<16><<<1, kIterThreads, 0, st>>>(P, range);
  else k_pm_iterate<kPmLocal><<<1, kIterThreads, 0, st>>>(P, range);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_pm_replan(const PlanDesc& P, uint32_t r, int shift, const float* x0_src, hipStream_t st) {
  if (P.K <= kPmChunk) return launch_range(P, r, shift, x0_src, P.K, WholeReplan{}, st);
  for (int k0 = 0; k0 < P.K; k0 += kPmChunk) {
    const int k1 = std::min(k0 + kPmChunk, P.K);
    // the caller's start state is read by the first kernel only, which keeps a copy
    const float* x0 = k0 == 0 ? x0_src : P.x0;
    const hipError_t e = launch_range(P, r, shift, x0, k1 - k0, IterRange{k0, k1}, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace mtp
