// A tile of point-mass rollouts: integrate first, then all cost terms at once.
//
// The double integrator's state is two dependent multiply-adds per step and
// dimension, while a step's cost (a test per obstacle) depends on that step's
// state alone.  A tile of C candidates therefore integrates on 2 C lanes,
// leaving the positions in LDS, takes the cost terms of all its (candidate,
// step) points with every thread of the workgroup, and adds them in step order
// on C lanes.  Every operation is the one-lane rollout's on the same operands
// (obstacle groups o mod 8 in increasing o, the groups in the same tree, the
// terms in step order), so the costs are the same bits.
#pragma once

#include "mtp_device.hpp"

namespace mtp {

constexpr int kTileSteps = 64;   // steps of a tile held in LDS at a time
constexpr int kTileBlock = 8;    // steps per block of the serial passes

template <int C>
struct PmTile {
  float u[kTileSteps][2][C];   // controls
  float p[kTileSteps][2][C];   // positions after the step
  float c[kTileSteps][C];      // cost terms
};

// Obstacles in LDS (centre x, centre y, squared radius), padded to a multiple
// of four with radius^2 = -1 (never hit); returns the padded count.
__device__ __forceinline__ int load_obstacles(const PlanDesc& P, float4* obs) {
  const float* tk = P.task;
  const int n_obs = static_cast<int>(tk[5]);
  const int padded = (n_obs + 3) & ~3;
  for (int i = threadIdx.x; i < padded; i += blockDim.x) {
    float4 o{0.0f, 0.0f, -1.0f, 0.0f};
    if (i < n_obs) {
      const float r = tk[6 + 3 * i + 2];
      o = float4{tk[6 + 3 * i], tk[6 + 3 * i + 1], r * r, 0.0f};
    }
    obs[i] = o;
  }
  return padded;
}

// Costs of a tile of C candidates whose controls gen(t0, steps) writes to sm.u
// chunk by chunk; rec(t, dim, cand, pos, vel) sees every state.  Every thread
// of the workgroup (BS of them) calls this; the costs are returned on threads
// 0 .. C - 1.  R: (candidate, step) points per thread, all of a chunk's unless the
// horizon is shorter (pm_points).
template <int C, int BS>
constexpr int kPmPoints = kTileSteps * C / BS > 0 ? kTileSteps * C / BS : 1;
template <int C, int BS, int R = kPmPoints<C, BS>, class Gen, class Rec>
__device__ __forceinline__ float pm_tile_cost(const PlanDesc& P, PmTile<C>& sm, const float4* obs, int n_pad, Gen gen,
                                              Rec rec) {
  const int tid = threadIdx.x;
  const float* tk = P.task;
  const float gx = tk[0], gy = tk[1], wg = tk[2], pen = tk[3], wu = tk[4];
  const float dt = P.dt;
  const int dim = tid / C, cand = tid % C;
  float pos = 0.0f, vel = 0.0f, cost = 0.0f;
  if (tid < 2 * C) {
    pos = P.x0[dim];
    vel = P.x0[2 + dim];
  }
  for (int t0 = 0; t0 < P.T; t0 += kTileSteps) {
    const int steps = min(kTileSteps, P.T - t0);
    gen(t0, steps);
    __syncthreads();
    // both serial passes go by whole blocks of steps, the next block's values
    // loading while the current one's are used; the steps past the end of the
    // last block are integrated and ignored, and their cost terms are zero
    const int blocks = (steps + kTileBlock - 1) / kTileBlock;
    if (tid < 2 * C) {
      float cu[kTileBlock], nu[kTileBlock];
#pragma unroll
      for (int i = 0; i < kTileBlock; ++i) cu[i] = sm.u[i][dim][cand];
      for (int b = 0; b < blocks; ++b) {
        const int i0 = b * kTileBlock, i1 = min(b + 1, blocks - 1) * kTileBlock;
#pragma unroll
        for (int i = 0; i < kTileBlock; ++i) nu[i] = sm.u[i1 + i][dim][cand];
#pragma unroll
        for (int i = 0; i < kTileBlock; ++i) {
          vel = fmaf(dt, cu[i], vel);
          pos = fmaf(dt, vel, pos);
          sm.p[i0 + i][dim][cand] = pos;
          if (i0 + i < steps) rec(t0 + i0 + i, dim, cand, pos, vel);
        }
#pragma unroll
        for (int i = 0; i < kTileBlock; ++i) cu[i] = nu[i];
      }
    }
    __syncthreads();
    const int points = blocks * kTileBlock * C;
    if (tid < points) {
      float px[R], py[R], g[R][8];
#pragma unroll
      for (int q = 0; q < R; ++q) {
        const int i = min((tid + q * BS) / C, kTileSteps - 1), c = (tid + q * BS) % C;
        px[q] = sm.p[i][0][c];
        py[q] = sm.p[i][1][c];
#pragma unroll
        for (int o = 0; o < 8; ++o) g[q][o] = 0.0f;
      }
      auto four = [&](int o0, auto half) {
#pragma unroll
        for (int o = 0; o < 4; ++o) {
          const float4 ob = obs[o0 + o];
#pragma unroll
          for (int q = 0; q < R; ++q) {
            const float ox = px[q] - ob.x, oy = py[q] - ob.y;
            g[q][4 * decltype(half)::value + o] += (fmaf(ox, ox, oy * oy) < ob.z) ? pen : 0.0f;
          }
        }
      };
      for (int o0 = 0; o0 < n_pad; o0 += 8) {
        four(o0, std::integral_constant<int, 0>{});
        if (o0 + 4 < n_pad) four(o0 + 4, std::integral_constant<int, 1>{});
      }
#pragma unroll
      for (int q = 0; q < R; ++q) {
        const int at = tid + q * BS;
        if (at < points) {
          const int i = at / C, c = at % C;
          const float obst = ((g[q][0] + g[q][1]) + (g[q][2] + g[q][3])) + ((g[q][4] + g[q][5]) + (g[q][6] + g[q][7]));
          const float dx = px[q] - gx, dy = py[q] - gy;
          const float ux = sm.u[i][0][c], uy = sm.u[i][1][c];
          float v = fmaf(wg, fmaf(dx, dx, dy * dy), obst);
          v = fmaf(wu, fmaf(ux, ux, uy * uy), v);
          sm.c[i][c] = i < steps ? v : 0.0f;
        }
      }
    }
    __syncthreads();
    if (tid < C) {
      float cc[kTileBlock], nc[kTileBlock];
#pragma unroll
      for (int i = 0; i < kTileBlock; ++i) cc[i] = sm.c[i][tid];
      for (int b = 0; b < blocks; ++b) {
        const int i1 = min(b + 1, blocks - 1) * kTileBlock;
#pragma unroll
        for (int i = 0; i < kTileBlock; ++i) nc[i] = sm.c[i1 + i][tid];
#pragma unroll
        for (int i = 0; i < kTileBlock; ++i) cost += cc[i];
#pragma unroll
        for (int i = 0; i < kTileBlock; ++i) cc[i] = nc[i];
      }
    }
  }
  return finite_or_inf(cost);
}

}  // namespace mtp
