// Wide rollout forms: more lanes per candidate than the one-lane and pair-lane
// forms of mtp_device.hpp, for launches that would leave most of the chip idle.
//
// What bounds such a launch is one wave's time through the horizon: the number
// of instructions a lane issues per step and the serial chain of the tension
// solve.  Here the links of a chain are spread over 2..8 lanes, so everything
// but that chain is divided by the lane count; the chain itself (elimination,
// back substitution, node position sums) keeps its order and runs segment by
// segment: every lane walks its rows once per segment, taking the carry of the
// lane before it, and the lane of segment g holds the right values from pass g
// on (a pass with the right carry reproduces them).  The passes issue as many
// row instructions as the narrow form, and every operation is the narrow
// form's on the same operands, so a wide form returns the same bits.
#pragma once

#include "mtp_device.hpp"

namespace mtp {

// ------------------------------------------------------------------ lane moves
template <int CTRL, int BANKS = 0xF>
__device__ __forceinline__ float dpp_move(float old, float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(v), CTRL, 0xF, BANKS, true));
}

// Moves among the 2 S lanes [A0 .. A(S-1) B0 .. B(S-1)] of a candidate whose
// halves A (base) and B (tip) meet at segment S - 1.  prev: segment g - 1 to g
// (the first one reads itself); next: g + 1 to g (the last one reads itself);
// swap: the two innermost segments exchange; inner: segment S - 1 to every
// segment of its half.  No move leaves the candidate, so a value that a caller
// multiplies by zero is never another candidate's.  A move is made by all lanes
// and its result selected afterwards: inside a conditional expression only some
// lanes would be active, and the others' values would read as zero.
template <int S>
struct HalfMoves;
template <>
struct HalfMoves<1> {
  static __device__ __forceinline__ float prev(float v) { return v; }
  static __device__ __forceinline__ float next(float v) { return v; }
  static __device__ __forceinline__ float swap(float v) { return pswap(v); }
  static __device__ __forceinline__ float inner(float v) { return v; }
};
template <>
struct HalfMoves<2> {
  static __device__ __forceinline__ float prev(float v) { return qperm<qperm_ctrl(0, 0, 2, 2)>(v); }
  static __device__ __forceinline__ float next(float v) { return qperm<qperm_ctrl(1, 1, 3, 3)>(v); }
  static __device__ __forceinline__ float swap(float v) { return qperm<qperm_ctrl(0, 3, 2, 1)>(v); }
  static __device__ __forceinline__ float inner(float v) { return qperm<qperm_ctrl(1, 1, 3, 3)>(v); }
};
template <>
struct HalfMoves<4> {   // each half is a quad
  static __device__ __forceinline__ float prev(float v) { return qperm<qperm_ctrl(0, 0, 1, 2)>(v); }
  static __device__ __forceinline__ float next(float v) { return qperm<qperm_ctrl(1, 2, 3, 3)>(v); }
  static __device__ __forceinline__ float swap(float v) {
    // half A (banks 0, 2 of a row) reads four lanes up, half B four lanes down
    return dpp_move<0x114, 0xA>(dpp_move<0x104, 0x5>(0.0f, v), v);
  }
  static __device__ __forceinline__ float inner(float v) { return qperm<qperm_ctrl(3, 3, 3, 3)>(v); }
};

// ------------------------------------------------------------------ two halves, S lanes each
// The pair-lane form with each half's N / 2 links cut into S segments of C.

template <int N, int S, bool EQ>
struct HalfConsts {
  static constexpr int C = N / (2 * S);
  float l[EQ ? 1 : C], invl[EQ ? 1 : C];
  __device__ __forceinline__ float len(int i) const { return l[EQ ? 0 : i]; }
  __device__ __forceinline__ float ilen(int i) const { return invl[EQ ? 0 : i]; }
  float im[C + 1];       // inverse masses of the segment's nodes
  float imb;             // im[0], the coupling to the segment before; 0 on a half's first segment
  float cont;            // 0 on a half's first segment, 1 elsewhere
  float half, bf, g0, sgn;
  float yg, kc, dc, ks, muf;
  bool B, outer, inner;  // tip half; first segment; last segment
  int seg;
};

template <int N, int S>
struct HalfTorque {
  static constexpr int C = N / (2 * S);
  float qa[C], qb[C], qc[C];
};

template <int N, int S, bool EQ>
__device__ __forceinline__ int half_link(const HalfConsts<N, S, EQ>& K, int i) {
  return pair_link<N>(K.B, K.seg * HalfConsts<N, S, EQ>::C + i);
}

template <int N, int S, bool EQ>
__device__ __forceinline__ void half_load_masses(const float* m, HalfConsts<N, S, EQ>& K) {
  constexpr int C = N / (2 * S);
#pragma unroll
  for (int i = 0; i <= C; ++i) {
    const int node = K.seg * C + i;
    const bool base = node == 0 && !K.B;
    const float mass = m[base ? 0 : pair_node_mass<N>(K.B, node)];
    K.im[i] = base ? 0.0f : 1.0f / mass;
  }
  K.imb = K.outer ? 0.0f : K.im[0];
}

// pair_solve on a segment: see there for the equations.  dFx, dFy: relative
// acceleration of each link's two nodes.
template <int N, int S, bool FORCES, bool EQ>
__device__ __forceinline__ void half_solve(const float (&s)[N / (2 * S)], const float (&c)[N / (2 * S)],
                                           const float (&w)[N / (2 * S)], const HalfTorque<N, S>& Q,
                                           const HalfConsts<N, S, EQ>& K, float so, float co,
                                           const float (&dFx)[N / (2 * S)], const float (&dFy)[N / (2 * S)],
                                           float (&acc)[N / (2 * S)]) {
  constexpr int C = N / (2 * S);
  using Mv = HalfMoves<S>;
  float P[C], X[C];   // cos and sin of phi_i - phi_{i+1}
#pragma unroll
  for (int i = 0; i < C; ++i) {
    const float sn = (i + 1 < C) ? s[i + 1] : so, cn = (i + 1 < C) ? c[i + 1] : co;
    P[i] = fmaf(c[i], cn, s[i] * sn);
    X[i] = fmaf(s[i], cn, -c[i] * sn);
  }
  // the coupling to the segment before (its coefficients are zero on a half's first)
  const float Pb = Mv::prev(P[C - 1]), Xb = Mv::prev(X[C - 1]);
  float Lp[C], Up[C], rhs[C];
#pragma unroll
  for (int i = 0; i < C; ++i) {
    float r = K.len(i) * w[i] * w[i];
    if constexpr (FORCES) {
      r = fmaf(s[i], dFx[i], r);
      r = fmaf(-c[i], dFy[i], r);
    } else if (i == 0) {
      r = fmaf(-c[0], -K.g0, r);
    }
    r = fmaf(Q.qa[i], X[i], r);
    r = fmaf(Q.qb[i], i > 0 ? X[i - 1] : Xb, r);
    rhs[i] = r;
    Lp[i] = i > 0 ? -K.im[i] * P[i - 1] : -K.imb * Pb;
    Up[i] = -K.im[i + 1] * P[i];
  }
  float cp[C], dp[C];
#pragma unroll
  for (int g = 0; g < S; ++g) {
    float cpv = 0.0f, dpv = 0.0f;
    if (g > 0) {
      cpv = Mv::prev(cp[C - 1]);
      dpv = Mv::prev(dp[C - 1]);
    }
#pragma unroll
    for (int i = 0; i < C; ++i) {
      const float inv = __builtin_amdgcn_rcpf(fmaf(-Lp[i], cpv, K.im[i] + K.im[i + 1]));
      cpv = Up[i] * inv;
      dpv = fmaf(-Lp[i], dpv, rhs[i]) * inv;
      cp[i] = cpv;
      dp[i] = dpv;
    }
  }
  // the two middle unknowns (right on the inner segments), then outwards
  float T[C];
  {
    const float cpo = Mv::swap(cp[C - 1]), dpo = Mv::swap(dp[C - 1]);
    const float mid = fmaf(-cp[C - 1], dpo, dp[C - 1]) * __builtin_amdgcn_rcpf(fmaf(-cp[C - 1], cpo, 1.0f));
    float last = mid;
#pragma unroll
    for (int g = 0; g < S; ++g) {
      if (g > 0) {
        const float tn = Mv::next(T[0]);
        last = K.inner ? mid : fmaf(-cp[C - 1], tn, dp[C - 1]);
      }
      T[C - 1] = last;
#pragma unroll
      for (int i = C - 2; i >= 0; --i) T[i] = fmaf(-cp[i], T[i + 1], dp[i]);
    }
  }
  const float T_sw = Mv::swap(T[C - 1]), T_nx = Mv::next(T[0]), Tb = Mv::prev(T[C - 1]);
  const float To = K.inner ? T_sw : T_nx;
#pragma unroll
  for (int i = 0; i < C; ++i) {
    float a = fmaf(Q.qa[i], P[i], Q.qc[i]);
    a = fmaf(-K.im[i + 1] * ((i + 1 < C) ? T[i + 1] : To), X[i], a);
    a = fmaf(-Q.qb[i], i > 0 ? P[i - 1] : Pb, a);
    a = fmaf(i > 0 ? K.im[i] * T[i - 1] : K.imb * Tb, i > 0 ? X[i - 1] : Xb, a);
    if constexpr (FORCES) {
      a = fmaf(c[i], dFx[i], fmaf(s[i], dFy[i], a));
    } else if (i == 0) {
      a = fmaf(s[0], -K.g0, a);
    }
    acc[i] = a * K.ilen(i);
  }
}

// pair_accel on a segment.
template <int N, int S, bool CONTACT, bool EQ>
__device__ __forceinline__ void half_accel(const float (&s)[N / (2 * S)], const float (&c)[N / (2 * S)],
                                           const float (&w)[N / (2 * S)], const HalfTorque<N, S>& Q,
                                           const HalfConsts<N, S, EQ>& K, float (&acc)[N / (2 * S)]) {
  constexpr int C = N / (2 * S);
  using Mv = HalfMoves<S>;
  // the next link's direction: the following segment's first, or the other
  // half's innermost one in this half's (reversed) frame
  const float s_sw = Mv::swap(s[C - 1]), c_sw = Mv::swap(c[C - 1]);
  const float s_nx = Mv::next(s[0]), c_nx = Mv::next(c[0]);
  const float so = K.inner ? -s_sw : s_nx, co = K.inner ? -c_sw : c_nx;
  float dFx[C], dFy[C];
  if constexpr (CONTACT) {
    float py[C + 1];
#pragma unroll
    for (int g = 0; g < S; ++g) {
      py[0] = g > 0 ? K.cont * Mv::prev(py[C]) : 0.0f;
#pragma unroll
      for (int i = 0; i < C; ++i) py[i + 1] = fmaf(-K.len(i), c[i], py[i]);
    }
    const float y0 = Mv::inner(K.bf * (Mv::swap(py[C]) - py[C]));
    float lowest = py[0];
#pragma unroll
    for (int i = 1; i <= C; ++i) lowest = fminf(lowest, py[i]);
    if (__builtin_amdgcn_ballot_w64(lowest + y0 < K.yg) != 0) {
      float vx[C + 1], vy[C + 1];
#pragma unroll
      for (int g = 0; g < S; ++g) {
        vx[0] = g > 0 ? K.cont * Mv::prev(vx[C]) : 0.0f;
        vy[0] = g > 0 ? K.cont * Mv::prev(vy[C]) : 0.0f;
#pragma unroll
        for (int i = 0; i < C; ++i) {
          const float lw = K.len(i) * w[i];
          vx[i + 1] = fmaf(lw, c[i], vx[i]);
          vy[i + 1] = fmaf(lw, s[i], vy[i]);
        }
      }
      const float u0 = Mv::inner(K.bf * (Mv::swap(vx[C]) - vx[C]));
      const float v0 = Mv::inner(K.bf * (Mv::swap(vy[C]) - vy[C]));
      const float ygl = K.yg - y0, dv0 = -K.dc * v0, ku0 = K.ks * u0;
      const float mu2 = 2.0f * K.muf, nmu = -K.muf;
      // Node accelerations as in pair_accel.  Its differences between
      // neighbouring nodes are contracted by the compiler: the product of one
      // of the two nodes goes into the fused operation, the farther node's, but
      // the nearer one's for Fx at a half's first link and for Fy at the even
      // ones after it; here that is written out, so the lane forms round alike
      // (written out in pair_accel too it cost the batched launch 3 to 5 %; another
      // compiler may contract that form otherwise, which the tests would show).
      float fn[C + 1], fr[C + 1], Fx[C + 1], Fy[C + 1];
#pragma unroll
      for (int i = 0; i <= C; ++i) {
        const float pen = ygl - py[i];
        fn[i] = pen > 0.0f ? fmaxf(fmaf(K.kc, pen, fmaf(-K.dc, vy[i], dv0)), 0.0f) : 0.0f;
        fr[i] = fmaf(mu2, __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(fmaf(K.ks, vx[i], ku0))), nmu);
        Fy[i] = fn[i] * K.im[i];
        Fx[i] = Fy[i] * fr[i];
      }
      const float edge = fmaf(-Fy[0], fr[0], Fx[1]);
#pragma unroll
      for (int i = 0; i < C; ++i) {
        dFx[i] = fmaf(Fy[i + 1], fr[i + 1], -Fx[i]);
        const float near = fmaf(-fn[i], K.im[i], Fy[i + 1]);
        const float far = fmaf(fn[i + 1], K.im[i + 1], -(i == 0 ? fmaf(fn[0], K.im[0], K.g0) : Fy[i]));
        const int place = K.seg * C + i;
        dFy[i] = (C % 2 == 0 && i > 0 ? i % 2 == 0 : place % 2 == 0 && place > 0) ? near : far;
      }
      dFx[0] = K.outer ? edge : dFx[0];
      half_solve<N, S, true>(s, c, w, Q, K, so, co, dFx, dFy, acc);
      return;
    }
  }
  half_solve<N, S, false>(s, c, w, Q, K, so, co, dFx, dFy, acc);
}

// Cost of candidate b under randomised model rep, on the group's 2 S lanes
// (`pos`: lane within the group); the value is right on the lanes of the last
// segment (pos S - 1 among them).
template <int N, int S, bool CONTACT, bool EQ>
__device__ __forceinline__ float rollout_half(const PlanDesc& P, int b, int pos, int rep, bool live) {
  constexpr int C = N / (2 * S);
  using Mv = HalfMoves<S>;
  const float* tk = P.task;
  HalfConsts<N, S, EQ> K;
  K.B = pos >= S;
  K.seg = K.B ? pos - S : pos;
  K.outer = K.seg == 0;
  K.inner = K.seg == S - 1;
  const bool B = K.B;
  K.half = B ? 0.5f : 0.0f;
  K.bf = B ? 1.0f : 0.0f;
  K.cont = K.outer ? 0.0f : 1.0f;
  K.g0 = (B || !K.outer) ? 0.0f : tk[0];
  K.sgn = B ? -1.0f : 1.0f;
#pragma unroll
  for (int i = 0; i < (EQ ? 1 : C); ++i) {
    K.l[i] = tk[5 + N + half_link(K, i)];
    K.invl[i] = 1.0f / K.l[i];
  }
  if constexpr (CONTACT) {
    K.yg = tk[5 + 2 * N]; K.kc = tk[6 + 2 * N]; K.dc = tk[7 + 2 * N];
    K.ks = 2.8853900817779268f * (1.0f / tk[8 + 2 * N]);
    const float* sp = P.sparams + (static_cast<size_t>(rep) * P.B + b) * (N + 1);
    half_load_masses<N, S>(sp, K);
    K.muf = sp[N];
  } else {
    half_load_masses<N, S>(tk + 5, K);
    K.ks = 0.0f; K.muf = 0.0f; K.yg = 0.0f; K.kc = 0.0f; K.dc = 0.0f;
  }
  const float wg = tk[1], wu = tk[2], tgx = tk[3], tgy = tk[4];
  const float dt = P.dt, hdt = 0.5f * P.dt, dt6 = P.dt * (1.0f / 6.0f);
  const float dtr = kInvTwoPi * dt, hdtr = kInvTwoPi * hdt, dt6r = kInvTwoPi * dt6;
  float ph[C], om[C], turn[C], s[C], c[C], hu[C];
#pragma unroll
  for (int i = 0; i < C; ++i) {
    const int k = half_link(K, i);
    const float r = fmaf(P.x0[k], kInvTwoPi, K.half);
    turn[i] = floorf(r);
    ph[i] = r - turn[i];
    om[i] = P.x0[N + k];
    rev_sincos_unit(ph[i], &s[i], &c[i], &hu[i]);
  }
  // controls through a buffer descriptor based at each step's block of U rows
  const uint32_t ldu = static_cast<uint32_t>(P.ldU);
  uint32_t uoff[C];
#pragma unroll
  for (int i = 0; i < C; ++i) uoff[i] = (static_cast<uint32_t>(half_link(K, i)) * ldu + static_cast<uint32_t>(b)) * 4u;
  const int step_bytes = static_cast<int>(static_cast<uint32_t>(N) * ldu * 4u);
  auto step_rows = [&](int t) {
    return __builtin_amdgcn_make_buffer_rsrc(P.U + static_cast<size_t>(t) * N * ldu, static_cast<short>(0), step_bytes,
                                             kBufferWord3);
  };
  float u[C];
  {
    const auto rs = step_rows(0);
#pragma unroll
    for (int i = 0; i < C; ++i) u[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, uoff[i], 0, 0));
  }
  float cost = 0.0f;
  const bool record = live && b < P.n_dbg;
  for (int t = 0; t < P.T; ++t) {
    float un[C];
    const int tn = (t + 1 < P.T) ? t + 1 : t;
    const auto rs = step_rows(tn);
#pragma unroll
    for (int i = 0; i < C; ++i) un[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, uoff[i], 0, 0));
    float q[C];
    const float u_sw = Mv::swap(u[C - 1]), u_nx = Mv::next(u[0]), u_pv = Mv::prev(u[C - 1]);
    const float u_next = K.inner ? u_sw : u_nx, u_prev = K.outer ? 0.0f : u_pv;
#pragma unroll
    for (int i = 0; i < C; ++i) {
      const float u_tip = B ? (i > 0 ? u[i - 1] : u_prev) : (i + 1 < C ? u[i + 1] : u_next);
      q[i] = (u[i] - u_tip) * K.ilen(i);
    }
    const float q_sw = Mv::swap(q[C - 1]), q_nx = Mv::next(q[0]), q_prev = Mv::prev(q[C - 1]);
    const float q_next = K.inner ? q_sw : q_nx;
    HalfTorque<N, S> Q;
#pragma unroll
    for (int i = 0; i < C; ++i) {
      Q.qa[i] = -K.im[i + 1] * ((i + 1 < C) ? q[i + 1] : q_next);
      Q.qb[i] = (i > 0) ? K.im[i] * q[i - 1] : K.imb * q_prev;
      Q.qc[i] = (K.im[i] + K.im[i + 1]) * q[i];
    }

    float kk[C], oms[C], aph[C], aom[C];
    half_accel<N, S, CONTACT>(s, c, om, Q, K, kk);
#pragma unroll
    for (int i = 0; i < C; ++i) {
      aph[i] = om[i];
      aom[i] = kk[i];
      oms[i] = om[i];
    }
#pragma unroll 1
    for (int stage = 1; stage < 4; ++stage) {
      const float h = (stage == 3) ? dt : hdt;
      const float hr = (stage == 3) ? dtr : hdtr;
      float s2[C], c2[C];
#pragma unroll
      for (int i = 0; i < C; ++i) {
        rev_sincos_scaled(fmaf(hr, oms[i], ph[i]), hu[i], &s2[i], &c2[i]);
        oms[i] = fmaf(h, kk[i], om[i]);
      }
      half_accel<N, S, CONTACT>(s2, c2, oms, Q, K, kk);
      const float wgt = (stage == 3) ? 1.0f : 2.0f;
#pragma unroll
      for (int i = 0; i < C; ++i) {
        aph[i] = fmaf(wgt, oms[i], aph[i]);
        aom[i] = fmaf(wgt, kk[i], aom[i]);
      }
    }
    float pu[C];
#pragma unroll
    for (int i = 0; i < C; ++i) {
      pu[i] = fmaf(dt6r, aph[i], ph[i]);
      ph[i] = __builtin_amdgcn_fractf(pu[i]);
      om[i] = fmaf(dt6, aom[i], om[i]);
      rev_sincos_unit(ph[i], &s[i], &c[i], &hu[i]);
    }
    // the half's link sums, outermost segment first
    float ex = 0.0f, ey = 0.0f, uu = 0.0f;
#pragma unroll
    for (int g = 0; g < S; ++g) {
      if (g > 0) {
        ex = K.cont * Mv::prev(ex);
        ey = K.cont * Mv::prev(ey);
        uu = K.cont * Mv::prev(uu);
      }
#pragma unroll
      for (int i = 0; i < C; ++i) {
        ex = fmaf(K.len(i), s[i], ex);
        ey = fmaf(-K.len(i), c[i], ey);
        uu = fmaf(u[i], u[i], uu);
      }
    }
    ex *= K.sgn;
    ey *= K.sgn;
    ex += Mv::swap(ex);
    ey += Mv::swap(ey);
    uu += Mv::swap(uu);
    const float dx = ex - tgx, dy = ey - tgy;
    cost += fmaf(wg, fmaf(dx, dx, dy * dy), wu * uu);
    if (record) {
      float* Xr = P.X + static_cast<size_t>(rep) * P.T * P.d * P.n_dbg + b;
      const size_t ldx = static_cast<size_t>(P.n_dbg);
#pragma unroll
      for (int i = 0; i < C; ++i) {
        const int k = half_link(K, i);
        turn[i] += floorf(pu[i]);
        Xr[(t * 2 * N + k) * ldx] = kTwoPi * ((turn[i] + ph[i]) - K.half);
        Xr[(t * 2 * N + N + k) * ldx] = om[i];
      }
    }
#pragma unroll
    for (int i = 0; i < C; ++i) u[i] = un[i];
  }
  return cost;
}

// ------------------------------------------------------------------ one half, L lanes
// The one-lane form (chain_accel) with its N links over L lanes of a quad, C
// each; links past the chain end have zero couplings, rate and acceleration.

template <int L>
struct QuadMoves {
  static_assert(L == 1 || L == 2 || L == 4, "lanes of a quad");
  static __device__ __forceinline__ float prev(float v) {
    if constexpr (L == 4) return qperm<qperm_ctrl(0, 0, 1, 2)>(v);
    if constexpr (L == 2) return qperm<qperm_ctrl(0, 0, 2, 2)>(v);
    return v;
  }
  static __device__ __forceinline__ float next(float v) {
    if constexpr (L == 4) return qperm<qperm_ctrl(1, 2, 3, 3)>(v);
    if constexpr (L == 2) return qperm<qperm_ctrl(1, 1, 3, 3)>(v);
    return v;
  }
};

template <int C>
struct LineConsts {
  float l[C], invl[C];    // padded links: length 0 and inverse length 0
  float im[C];            // inverse mass of the link's end node (0 past the end)
  float imU[C];           // the same where a next link exists, else 0
  float imP[C];           // inverse mass of the node before (0 at the base and past the end)
  float D[C], imS[C];     // im + imP; D is 1 past the end
  float g0;               // gravity on the base link
  float yg, kc, dc, inv_vs, muf;
  float cont;             // 0 on lane 0, 1 elsewhere
};

template <int L, int C, bool CONTACT>
__device__ __forceinline__ void line_accel(const float (&s)[C], const float (&c)[C], const float (&om)[C],
                                           const float (&q)[C], float q_next, float q_prev, const LineConsts<C>& K,
                                           float (&acc)[C]) {
  using Mv = QuadMoves<L>;
  const float so = Mv::next(s[0]), co = Mv::next(c[0]);
  float P[C], X[C];
#pragma unroll
  for (int i = 0; i < C; ++i) {
    const float sn = (i + 1 < C) ? s[i + 1] : so, cn = (i + 1 < C) ? c[i + 1] : co;
    P[i] = fmaf(c[i], cn, s[i] * sn);
    X[i] = fmaf(s[i], cn, -c[i] * sn);
  }
  const float Pb = Mv::prev(P[C - 1]), Xb = Mv::prev(X[C - 1]);
  // change of the non-constraint acceleration across each link
  float dfx[C], dfy[C];
  if constexpr (CONTACT) {
    float py[C];
    float e = 0.0f;
#pragma unroll
    for (int g = 0; g < L; ++g) {
      if (g > 0) e = K.cont * Mv::prev(py[C - 1]);
#pragma unroll
      for (int i = 0; i < C; ++i) {
        e = fmaf(-K.l[i], c[i], e);
        py[i] = e;
      }
    }
    float lowest = py[0];
#pragma unroll
    for (int i = 1; i < C; ++i) lowest = fminf(lowest, py[i]);
    float fx[C], fy[C];
#pragma unroll
    for (int i = 0; i < C; ++i) { fx[i] = 0.0f; fy[i] = 0.0f; }
    // one branch for the wave: some node of some lane below the ground
    if (__builtin_amdgcn_ballot_w64(K.yg - lowest > 0.0f) != 0) {
      float vx[C], vy[C];
      float ax = 0.0f, ay = 0.0f;
#pragma unroll
      for (int g = 0; g < L; ++g) {
        if (g > 0) {
          ax = K.cont * Mv::prev(vx[C - 1]);
          ay = K.cont * Mv::prev(vy[C - 1]);
        }
#pragma unroll
        for (int i = 0; i < C; ++i) {
          const float lw = K.l[i] * om[i];
          ax = fmaf(lw, c[i], ax);
          ay = fmaf(lw, s[i], ay);
          vx[i] = ax;
          vy[i] = ay;
        }
      }
#pragma unroll
      for (int i = 0; i < C; ++i) {
        const float pen = K.yg - py[i];
        const float fn = fmaxf(fmaf(K.kc, pen, -K.dc * vy[i]), 0.0f);
        const float ft = -K.muf * fn * fast_tanh(vx[i] * K.inv_vs);
        fx[i] = pen > 0.0f ? ft * K.im[i] : 0.0f;
        fy[i] = pen > 0.0f ? fn * K.im[i] : 0.0f;
      }
    }
    const float bx = K.cont * Mv::prev(fx[C - 1]), by = K.cont * Mv::prev(fy[C - 1]);
#pragma unroll
    for (int i = 0; i < C; ++i) {
      dfx[i] = fx[i] - (i > 0 ? fx[i - 1] : bx);
      dfy[i] = fy[i] - (i > 0 ? fy[i - 1] : by);
      if (i == 0) dfy[0] -= K.g0;
    }
  }
  float Lo[C], Up[C], rhs[C];
#pragma unroll
  for (int i = 0; i < C; ++i) {
    const float Xp = i > 0 ? X[i - 1] : Xb, qp = i > 0 ? q[i - 1] : q_prev, qn = i + 1 < C ? q[i + 1] : q_next;
    float r = K.l[i] * om[i] * om[i];
    if constexpr (CONTACT) {
      r = fmaf(s[i], dfx[i], r);
      r = fmaf(-c[i], dfy[i], r);
    } else if (i == 0) {
      r = fmaf(-c[0], -K.g0, r);
    }
    r = fmaf(-K.imU[i] * qn, X[i], r);
    r = fmaf(K.imP[i] * qp, Xp, r);
    rhs[i] = r;
    Up[i] = -K.imU[i] * P[i];
    Lo[i] = -K.imP[i] * (i > 0 ? P[i - 1] : Pb);
  }
  float cp[C], dp[C];
#pragma unroll
  for (int g = 0; g < L; ++g) {
    float cpv = 0.0f, dpv = 0.0f;
    if (g > 0) {
      cpv = Mv::prev(cp[C - 1]);
      dpv = Mv::prev(dp[C - 1]);
    }
#pragma unroll
    for (int i = 0; i < C; ++i) {
      const float inv = __builtin_amdgcn_rcpf(fmaf(-Lo[i], cpv, K.D[i]));
      cpv = Up[i] * inv;
      dpv = fmaf(-Lo[i], dpv, rhs[i]) * inv;
      cp[i] = cpv;
      dp[i] = dpv;
    }
  }
  // back substitution: the lane of the last segment starts from its own value
  // (its coupling is zero), the others from the next lane's first tension
  float T[C];
#pragma unroll
  for (int g = 0; g < L; ++g) {
    float tn = 0.0f;
    if (g > 0) tn = Mv::next(T[0]);
#pragma unroll
    for (int i = C - 1; i >= 0; --i) {
      tn = fmaf(-cp[i], tn, dp[i]);
      T[i] = tn;
    }
  }
  const float To = Mv::next(T[0]), Tb = Mv::prev(T[C - 1]);
#pragma unroll
  for (int i = 0; i < C; ++i) {
    const float Xp = i > 0 ? X[i - 1] : Xb, Pp = i > 0 ? P[i - 1] : Pb;
    const float qp = i > 0 ? q[i - 1] : q_prev, qn = i + 1 < C ? q[i + 1] : q_next;
    float a = K.imS[i] * q[i];
    a = fmaf(-K.imU[i], fmaf(i + 1 < C ? T[i + 1] : To, X[i], qn * P[i]), a);
    a = fmaf(-K.imP[i], fmaf(-(i > 0 ? T[i - 1] : Tb), Xp, qp * Pp), a);
    if constexpr (CONTACT) {
      a += fmaf(c[i], dfx[i], s[i] * dfy[i]);
    } else if (i == 0) {
      a = fmaf(-K.g0, s[0], a);
    }
    acc[i] = a * K.invl[i];
  }
}

// Cost of candidate b under randomised model rep on the L lanes of a group;
// right on the group's last lane.
template <int N, int L, bool CONTACT>
__device__ __forceinline__ float rollout_line(const PlanDesc& P, int b, int pos, int rep, bool live) {
  constexpr int C = (N + L - 1) / L;
  using Mv = QuadMoves<L>;
  const float* tk = P.task;
  const float wg = tk[1], wu = tk[2], tx = tk[3], ty = tk[4];
  LineConsts<C> K;
  K.cont = pos == 0 ? 0.0f : 1.0f;
  K.g0 = pos == 0 ? tk[0] : 0.0f;
  const float* m = tk + 5;
  if constexpr (CONTACT) {
    K.yg = tk[5 + 2 * N]; K.kc = tk[6 + 2 * N]; K.dc = tk[7 + 2 * N]; K.inv_vs = 1.0f / tk[8 + 2 * N];
    m = P.sparams + (static_cast<size_t>(rep) * P.B + b) * (N + 1);
    K.muf = m[N];
  } else {
    K.muf = 0.0f; K.yg = 0.0f; K.kc = 0.0f; K.dc = 0.0f; K.inv_vs = 0.0f;
  }
  const float dt = P.dt, hdt = 0.5f * P.dt, dt6 = P.dt * (1.0f / 6.0f);
  const float dtr = kInvTwoPi * dt, hdtr = kInvTwoPi * hdt, dt6r = kInvTwoPi * dt6;
  float ph[C], om[C], turn[C], s[C], c[C], live_link[C];
  int link[C];
#pragma unroll
  for (int i = 0; i < C; ++i) {
    const int k = pos * C + i;
    const bool on = k < N;
    link[i] = on ? k : N - 1;
    live_link[i] = on ? 1.0f : 0.0f;
    const float len = tk[5 + N + link[i]];
    K.l[i] = on ? len : 0.0f;
    K.invl[i] = on ? 1.0f / len : 0.0f;
    const float im = on ? 1.0f / m[link[i]] : 0.0f;
    const float imp = (on && k > 0) ? 1.0f / m[k > 0 ? link[i] - 1 : 0] : 0.0f;
    K.im[i] = im;
    K.imU[i] = k + 1 < N ? im : 0.0f;
    K.imP[i] = imp;
    K.imS[i] = im + imp;
    K.D[i] = on ? im + imp : 1.0f;
    const float r = kInvTwoPi * P.x0[link[i]];
    turn[i] = floorf(r);
    ph[i] = on ? r - turn[i] : 0.0f;
    om[i] = on ? P.x0[N + link[i]] : 0.0f;
    rev_sincos(ph[i], &s[i], &c[i]);
  }
  const size_t ld = static_cast<size_t>(P.ldU);
  const float* ub = P.U + b;
  float u[C];
#pragma unroll
  for (int i = 0; i < C; ++i) u[i] = live_link[i] * ub[link[i] * ld];
  float cost = 0.0f;
  const bool record = live && b < P.n_dbg;
  for (int t = 0; t < P.T; ++t) {
    float un[C];
    const int tn = (t + 1 < P.T) ? t + 1 : t;
#pragma unroll
    for (int i = 0; i < C; ++i) un[i] = ub[(tn * N + link[i]) * ld];
    // torque differences over the links' lengths; u past the chain end is 0
    float q[C];
    const float u_nx = Mv::next(u[0]);
    const float u_next = pos == L - 1 ? 0.0f : u_nx;
#pragma unroll
    for (int i = 0; i < C; ++i) q[i] = (u[i] - (i + 1 < C ? u[i + 1] : u_next)) * K.invl[i];
    const float q_next = Mv::next(q[0]), q_prev = Mv::prev(q[C - 1]);

    float kk[C], oms[C], aph[C], aom[C];
    line_accel<L, C, CONTACT>(s, c, om, q, q_next, q_prev, K, kk);
#pragma unroll
    for (int i = 0; i < C; ++i) {
      aph[i] = om[i];
      aom[i] = kk[i];
      oms[i] = om[i];
    }
#pragma unroll 1
    for (int stage = 1; stage < 4; ++stage) {
      const float h = (stage == 3) ? dt : hdt;
      const float hr = (stage == 3) ? dtr : hdtr;
      float s2[C], c2[C];
#pragma unroll
      for (int i = 0; i < C; ++i) {
        rev_sincos(fmaf(hr, oms[i], ph[i]), &s2[i], &c2[i]);
        oms[i] = fmaf(h, kk[i], om[i]);
      }
      line_accel<L, C, CONTACT>(s2, c2, oms, q, q_next, q_prev, K, kk);
      const float wgt = (stage == 3) ? 1.0f : 2.0f;
#pragma unroll
      for (int i = 0; i < C; ++i) {
        aph[i] = fmaf(wgt, oms[i], aph[i]);
        aom[i] = fmaf(wgt, kk[i], aom[i]);
      }
    }
    float pu[C];
#pragma unroll
    for (int i = 0; i < C; ++i) {
      pu[i] = fmaf(dt6r, aph[i], ph[i]);
      ph[i] = __builtin_amdgcn_fractf(pu[i]);
      om[i] = fmaf(dt6, aom[i], om[i]);
      rev_sincos(ph[i], &s[i], &c[i]);
    }
    float ex = 0.0f, ey = 0.0f, uu = 0.0f;
#pragma unroll
    for (int g = 0; g < L; ++g) {
      if (g > 0) {
        ex = K.cont * Mv::prev(ex);
        ey = K.cont * Mv::prev(ey);
        uu = K.cont * Mv::prev(uu);
      }
#pragma unroll
      for (int i = 0; i < C; ++i) {
        ex = fmaf(K.l[i], s[i], ex);
        ey = fmaf(-K.l[i], c[i], ey);
        uu = fmaf(u[i], u[i], uu);
      }
    }
    const float dx = ex - tx, dy = ey - ty;
    cost += fmaf(wg, fmaf(dx, dx, dy * dy), wu * uu);
    if (record) {
      float* Xr = P.X + static_cast<size_t>(rep) * P.T * P.d * P.n_dbg + b;
      const size_t ldx = static_cast<size_t>(P.n_dbg);
#pragma unroll
      for (int i = 0; i < C; ++i) {
        turn[i] += floorf(pu[i]);
        if (live_link[i] != 0.0f) {
          Xr[(t * 2 * N + link[i]) * ldx] = kTwoPi * (turn[i] + ph[i]);
          Xr[(t * 2 * N + N + link[i]) * ldx] = om[i];
        }
      }
    }
#pragma unroll
    for (int i = 0; i < C; ++i) u[i] = live_link[i] * un[i];
  }
  return cost;
}

}  // namespace mtp
