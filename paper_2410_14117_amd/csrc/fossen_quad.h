// fossen_quad.h -- the control step of fossen_device.h with one env spread
// over a quad of four lanes, for launches too small to fill the GPU with one
// env per lane.
//
// A launch of few waves lasts as long as one wave's instruction chain: a lone
// wave issues one VALU instruction every 2.0-2.3 ns whatever its lanes hold
// (measured: 128 and 1024 one-wave blocks, FMA chains, dependent or not), and
// one env per lane puts 457 of them into a sub-step.  Here lane c of a quad
// holds component c of the quaternion (w, x, y, z) and, for c = 1..3, of each
// 3-vector (position, linear and angular velocity, momenta, residuals), so one
// instruction serves a whole vector and a cross product reads its rotated
// operands through DPP quad permutations.  Lane 0 carries finite don't-care
// values in the 3-vectors that no other lane reads.  241 instructions per
// sub-step, 1.9 times fewer; the total over the chip grows (four lanes do
// the work of one 1.9 times), which is why large launches keep one env per lane.
//
// Every value is formed by the same operations in the same order as in
// fossen_device.h (the per-component formulas there are cyclic in x, y, z), so
// results are equal, bitwise, up to the sign of zeros.  Contraction is off:
// every FMA is written out.  Thruster states and throttles: lane c holds
// thrusters c and c + 4.
#pragma once

#include "fossen_device.h"

namespace mg {

#pragma clang fp contract(off)

// lane i of each quad reads lane p_i
#define MG_QP(p0, p1, p2, p3) ((p0) | ((p1) << 2) | ((p2) << 4) | ((p3) << 6))
template <int CTRL>
__device__ __forceinline__ float qperm(float x) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ int qperm(int x) {
  return __builtin_amdgcn_mov_dpp(x, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ double qperm(double x) {
  const int64_t v = __builtin_bit_cast(int64_t, x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)v, CTRL, 0xf, 0xf, true);
  const uint32_t hi =
      (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(v >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, (int64_t)(((uint64_t)hi << 32) | lo));
}
constexpr int kRot1 = MG_QP(1, 2, 3, 1);    // component i + 1 of a 3-vector (lane 0: x)
constexpr int kRot2 = MG_QP(2, 3, 1, 2);    // component i + 2 (lane 0: y)
constexpr int kSwapXY = MG_QP(0, 2, 1, 3);  // x <-> y
constexpr int kQRot1 = MG_QP(2, 2, 3, 1);   // quaternion: component i + 1, lane 0: y
constexpr int kQRot2 = MG_QP(1, 3, 1, 2);   // component i + 2, lane 0: x
constexpr int kQW = MG_QP(3, 0, 0, 0);      // w, lane 0: z

// Lane constants that do not depend on the env.
struct QuadLane {
  float sg;          // -1 in lane 0, else 1
  float kc, kf, ke;  // factors of k = R^T e3 (quad_residual)
  int c;             // component
};
__device__ __forceinline__ QuadLane quad_lane(int lane) {
  QuadLane L;
  L.c = lane & 3;
  L.sg = L.c == 0 ? -1.0f : 1.0f;
  L.kc = (L.c & 1) ? -2.0f : 2.0f;               // x, y, z: -2, 2, -2
  L.kf = L.c == 3 ? -2.0f : 2.0f;                // x, y, z: 2, 2, -2
  L.ke = L.c == 3 ? 1.0f : 0.0f;
  return L;
}

// The env of a lane's quad: its class and internal column.  A quad with no env
// (past its class's envs, or in a block past the last) loads column 0, which
// every sim has, and stores nothing; the first column of its class need not
// exist, since a declared class may have no envs.
struct QuadEnv {
  int cls;
  bool active;   // all four lanes of a quad alike
  uint32_t j;
};
template <class ARGS>
__host__ __device__ __forceinline__ QuadEnv quad_env(const ARGS& a, const ClassSegs& segs, int b,
                                                     int lane) {
  QuadEnv e;
  int block;
  e.cls = block_class(segs, b, block);
  const int64_t start = segs.start[e.cls], len = segs.len[e.cls];
  const int64_t local = (int64_t)block * kQuadEnvs + (lane >> 2);
  e.active = local < len && MG_CHECK(a, start + len <= a.Ep, kDbgSegment);
  e.j = e.active ? (uint32_t)(start + local) : 0u;
  if (!MG_CHECK(a, (int64_t)e.j < a.Ep, kDbgInternal)) {   // also of quads with no env
    e.active = false;
    e.j = 0u;
  }
  return e;
}

// The state of one env: lane c's components.
struct QuadState {
  float p, q, v, w;   // position, quaternion, linear and angular velocity
  float f[2];         // thruster states c, c + 4
};

// The per-env constants a sub-step reads (lane c's components): the coupling
// terms sit in the x and y lanes, 0 elsewhere.
struct QuadConst {
  float Al, Aa, Acl, Aca;   // (h/2) M^-1: diagonal (lin, ang) and coupling
  float dll, dla, dql, dqa; // damping
  float wmb, hz;            // W - B;  (-h_z, h_z, 0)
};
// M itself, for the momentum at the start of a control step.
struct QuadMass {
  float l, a, cl, ca;
};

// C (c + 1 rows of the env's derived constants): row pointers are wave-uniform,
// j4 the env's byte offset, s4 the row stride in bytes.
__device__ __forceinline__ float quad_row(const float* base, uint32_t off) {
  return lane_elem(base, off);
}
__device__ __forceinline__ void load_quad_const(const float* der, int64_t Ep, uint32_t j4, int c,
                                                float h2, QuadConst& C, QuadMass& M) {
  const uint32_t s4 = (uint32_t)Ep * 4u;
  const uint32_t oi = j4 + (c > 1 ? (uint32_t)(c - 1) * s4 : 0u);
  const uint32_t sw = c == 2 ? s4 : 0u;
  const bool xy = c == 1 || c == 2;
  M.l = quad_row(der + kMuu * Ep, oi);
  M.a = quad_row(der + kMpp * Ep, oi);
  const float mcl = quad_row(der + kMuq * Ep, j4 + sw);
  const float mca = quad_row(der + kMuq * Ep, j4 + s4 - sw);
  const float il = quad_row(der + kIuu * Ep, oi);
  const float ia = quad_row(der + kIpp * Ep, oi);
  const float icl = quad_row(der + kIuq * Ep, j4 + sw);
  const float ica = quad_row(der + kIuq * Ep, j4 + s4 - sw);
  C.dll = quad_row(der + kDL * Ep, oi);
  C.dla = quad_row(der + (kDL + 3) * Ep, oi);
  C.dql = quad_row(der + kDQ * Ep, oi);
  C.dqa = quad_row(der + (kDQ + 3) * Ep, oi);
  C.wmb = quad_row(der + kWmB * Ep, j4);
  const float hz = quad_row(der + kHz * Ep, j4);
  C.hz = c == 1 ? -hz : (c == 2 ? hz : 0.0f);
  M.cl = xy ? mcl : 0.0f;
  M.ca = xy ? mca : 0.0f;
  C.Al = h2 * il;
  C.Aa = h2 * ia;
  C.Acl = xy ? h2 * icl : 0.0f;
  C.Aca = xy ? h2 * ica : 0.0f;
}

// One row (k < 3: lane c's linear, else angular) of the allocation matrix and
// the wave-uniform thruster data of the class.
struct QuadThr {
  float bl[kMaxThr], ba[kMaxThr];   // B[c - 1][i], B[c + 2][i]
  float f_max, rho_s;
  int n, map, lag;
};
__device__ __forceinline__ void load_quad_thr(const ClassConst* cc, int c, QuadThr& t) {
  const int i = c > 1 ? c - 1 : 0;
#pragma unroll
  for (int k = 0; k < kMaxThr; ++k) {
    t.bl[k] = cc->B[i][k];
    t.ba[k] = cc->B[3 + i][k];
  }
  t.f_max = cc->f_max;
  t.rho_s = cc->rho_s;
  t.n = cc->n_thr;
  t.map = cc->thr_map;
  t.lag = cc->lag;
}

// The lane's two thrusters, c and c + 4 of n, in rows of stride s4 bytes: offsets
// of loads (of row 0 past n, masked when the values are used, so that nothing
// branches and no load is waited for before the next one is issued).
struct QuadPair {
  uint32_t o0, o1;
  bool m0, m1;
};
__device__ __forceinline__ QuadPair quad_pair(int c, int n, uint32_t col, uint32_t s4) {
  QuadPair r;
  r.m0 = c < n;
  r.m1 = c + 4 < n;
  r.o0 = col + (r.m0 ? (uint32_t)c * s4 : 0u);
  r.o1 = col + (r.m1 ? (uint32_t)(c + 4) * s4 : 0u);
  return r;
}
__device__ __forceinline__ void quad_load_pair(const QuadPair& r, const float* rows,
                                               float (&v)[2]) {
  v[0] = lane_elem(rows, r.o0);
  v[1] = lane_elem(rows, r.o1);
}
__device__ __forceinline__ void quad_mask_pair(const QuadPair& r, float (&v)[2]) {
  v[0] = r.m0 ? v[0] : 0.0f;
  v[1] = r.m1 ? v[1] : 0.0f;
}
__device__ __forceinline__ void quad_store_pair(const QuadPair& r, float* rows,
                                                const float (&v)[2]) {
  if (r.m0) lane_elem(rows, r.o0) = v[0];
  if (r.m1) lane_elem(rows, r.o1) = v[1];
}

// clamp and thrust map of the lane's two throttles (thrust_command)
__device__ __forceinline__ void quad_thrust(const QuadThr& t, const float (&a)[2],
                                            float (&fcmd)[2]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const float ai = a[h] > 1.0f ? 1.0f : (a[h] < -1.0f ? -1.0f : a[h]);
    const float f = t.f_max * ai;
    fcmd[h] = t.map ? f * fabsf(ai) : f;
  }
}

// (l, a) = B f, thrusters in order (command_wrench, lag_wrench); those past the
// class's own are zeros with zero columns
__device__ __forceinline__ void quad_wrench(const QuadThr& t, const float (&f)[2], float& l,
                                            float& a) {
#define MG_BC(i) \
  qperm<MG_QP((i) & 3, (i) & 3, (i) & 3, (i) & 3)>(f[(i) >> 2])
  const float f0 = MG_BC(0);
  l = t.bl[0] * f0;
  a = t.ba[0] * f0;
#define MG_ACC(i)                 \
  {                               \
    const float fi = MG_BC(i);    \
    l = fmaf(t.bl[i], fi, l);     \
    a = fmaf(t.ba[i], fi, a);     \
  }
  MG_ACC(1) MG_ACC(2) MG_ACC(3) MG_ACC(4) MG_ACC(5) MG_ACC(6) MG_ACC(7)
#undef MG_ACC
#undef MG_BC
}

// Kinematic rates of a quad: kp = R(q) v, kq = q (x) (0, w) (TWICE q').
__device__ __forceinline__ void quad_kinematics(const QuadLane& L, float q, float v, float w,
                                                float& kp, float& kq) {
  const float q0 = qperm<kQW>(q), q1 = qperm<kQRot1>(q), q2 = qperm<kQRot2>(q);
  const float v1 = qperm<kRot1>(v), v2 = qperm<kRot2>(v);
  // lane 0 takes these two with a minus (q' of the scalar part); the other
  // lanes' second one is the component i + 2 of w
  const float w0 = qperm<MG_QP(3, 1, 2, 3)>(w) * L.sg, w2 = qperm<kRot2>(w) * L.sg;
  // t = 2 q_v x v
  const float th = fmaf(q1, v2, -(q2 * v1)), t = th + th;
  kp = fmaf(-q2, qperm<kRot1>(t), fmaf(q1, qperm<kRot2>(t), fmaf(q0, t, v)));
  kq = fmaf(-q2, qperm<kRot1>(w), fmaf(q1, w2, q0 * w0));
}

// The residual (rl, ra) of rhs_residual_m for a quad: the state (q, v, w) with
// momentum (ml, ma) and wrench (tl, ta).
__device__ __forceinline__ void quad_forces(const QuadLane& L, const QuadConst& C, float q,
                                            float v, float w, float ml, float ma, float tl,
                                            float ta, float& rl, float& ra) {
  const float v1 = qperm<kRot1>(v), v2 = qperm<kRot2>(v);
  const float w1 = qperm<kRot1>(w), w2 = qperm<kRot2>(w) * L.sg;
  // k = R^T e3: x (2 qx) qz - (2 qy) qw, y (2 qy) qz + (2 qx) qw,
  //             z 1 - (2 qx) qx - (2 qy) qy
  const float k = fmaf(qperm<MG_QP(3, 3, 3, 2)>(q), qperm<MG_QP(0, 1, 2, 2)>(q) * L.kf,
                       fmaf(qperm<MG_QP(0, 0, 0, 1)>(q), qperm<MG_QP(0, 2, 1, 1)>(q) * L.kc, L.ke));
  const float a1 = qperm<kRot1>(ml), a2 = qperm<kRot2>(ml);
  const float el = fmaf(C.dql, fabsf(v), C.dll), ea = fmaf(C.dqa, fabsf(w), C.dla);
  rl = fmaf(-el, v, fmaf(C.wmb, k, fmaf(-w1, a2, fmaf(w2, a1, tl))));
  ra = fmaf(-v1, a2, ta);
  ra = fmaf(v2, a1, ra);
  ra = fmaf(-w1, qperm<kRot2>(ma), ra);
  ra = fmaf(w2, qperm<kRot1>(ma), ra);
  ra = fmaf(qperm<kSwapXY>(k), C.hz, ra);
  ra = fmaf(-ea, w, ra);
}

// rhs_residual_m for a quad
__device__ __forceinline__ void quad_residual(const QuadLane& L, const QuadConst& C, float q,
                                              float v, float w, float ml, float ma, float tl,
                                              float ta, float& kp, float& kq, float& rl,
                                              float& ra) {
  quad_kinematics(L, q, v, w, kp, kq);
  quad_forces(L, C, q, v, w, ml, ma, tl, ta, rl, ra);
}

// (l, a) = base + A r (add_inv)
__device__ __forceinline__ void quad_add_inv(const QuadConst& C, float rl, float ra, float bl,
                                             float ba, float& l, float& a) {
  l = fmaf(C.Al, rl, fmaf(qperm<kSwapXY>(ra), C.Acl, bl));
  a = fmaf(C.Aa, ra, fmaf(qperm<kSwapXY>(rl), C.Aca, ba));
}
// (l, a) = A r (mul_inv)
__device__ __forceinline__ void quad_mul_inv(const QuadConst& C, float rl, float ra, float& l,
                                             float& a) {
  l = fmaf(C.Al, rl, qperm<kSwapXY>(ra) * C.Acl);
  a = fmaf(C.Aa, ra, qperm<kSwapXY>(rl) * C.Aca);
}

// Uniform RK4 factors in vector registers (an operand from a scalar register
// costs nothing in a lone wave, but the same code runs several waves to a SIMD).
struct QuadStep {
  float h2, h2q, dt, dtq, h6, h6q, third;
  float s2, s3, s4, rho;
};
__device__ __forceinline__ QuadStep quad_step_const(const ClassConst* cc, float dt) {
  QuadStep k;
  const float h2 = 0.5f * dt, h6 = dt * (1.0f / 6.0f);
  k.h2 = to_vgpr(h2);
  k.h2q = to_vgpr(0.5f * h2);
  k.dt = to_vgpr(dt);
  k.dtq = to_vgpr(0.5f * dt);
  k.h6 = to_vgpr(h6);
  k.h6q = to_vgpr(0.5f * h6);
  k.third = to_vgpr(1.0f / 3.0f);
  k.s2 = to_vgpr(cc->sigma2);
  k.s3 = to_vgpr(cc->sigma3);
  k.s4 = to_vgpr(cc->sigma4);
  k.rho = to_vgpr(cc->rho);
  return k;
}

// q <- q / |q| with the sum of squares in rk4_substep's order
__device__ __forceinline__ float quad_normalise(float q) {
  const float bw = qperm<MG_QP(0, 0, 0, 0)>(q), bx = qperm<MG_QP(1, 1, 1, 1)>(q);
  const float by = qperm<MG_QP(2, 2, 2, 2)>(q), bz = qperm<MG_QP(3, 3, 3, 3)>(q);
  return q * rsqrt_t(fmaf(bz, bz, fmaf(by, by, fmaf(bw, bw, bx * bx))));
}

// rk4_substep for a quad: (ml, ma) the carried momentum, (gl, ga) the command
// wrench, (dl, da) the carried lag wrench.
template <bool LAG>
__device__ __forceinline__ void quad_substep(const QuadLane& L, const QuadConst& C,
                                             const QuadStep& s, QuadState& x, float& ml, float& ma,
                                             float gl, float ga, float& dl, float& da) {
  float kp, kq, rl, ra, pp, pq, pl, pa, X, V, W, sl, sa;
  float tl = gl, ta = ga;
  if constexpr (LAG) {
    tl = gl + dl;
    ta = ga + da;
  }
  quad_residual(L, C, x.q, x.v, x.w, ml, ma, tl, ta, kp, kq, rl, ra);
  pp = kp; pq = kq; pl = rl; pa = ra;
  X = fmaf(s.h2q, kq, x.q);
  sl = fmaf(s.h2, rl, ml);
  sa = fmaf(s.h2, ra, ma);
  quad_add_inv(C, rl, ra, x.v, x.w, V, W);
  if constexpr (LAG) {
    tl = fmaf(s.s2, dl, gl);
    ta = fmaf(s.s2, da, ga);
  }
  quad_residual(L, C, X, V, W, sl, sa, tl, ta, kp, kq, rl, ra);
  pp = fmaf(2.0f, kp, pp); pq = fmaf(2.0f, kq, pq);
  pl = fmaf(2.0f, rl, pl); pa = fmaf(2.0f, ra, pa);
  X = fmaf(s.h2q, kq, x.q);
  sl = fmaf(s.h2, rl, ml);
  sa = fmaf(s.h2, ra, ma);
  quad_add_inv(C, rl, ra, x.v, x.w, V, W);
  if constexpr (LAG) {
    tl = fmaf(s.s3, dl, gl);
    ta = fmaf(s.s3, da, ga);
  }
  quad_residual(L, C, X, V, W, sl, sa, tl, ta, kp, kq, rl, ra);
  pp = fmaf(2.0f, kp, pp); pq = fmaf(2.0f, kq, pq);
  pl = fmaf(2.0f, rl, pl); pa = fmaf(2.0f, ra, pa);
  X = fmaf(s.dtq, kq, x.q);
  sl = fmaf(s.dt, rl, ml);
  sa = fmaf(s.dt, ra, ma);
  float yl, ya;
  quad_mul_inv(C, rl, ra, yl, ya);
  V = fmaf(2.0f, yl, x.v);
  W = fmaf(2.0f, ya, x.w);
  if constexpr (LAG) {
    tl = fmaf(s.s4, dl, gl);
    ta = fmaf(s.s4, da, ga);
  }
  quad_residual(L, C, X, V, W, sl, sa, tl, ta, kp, kq, rl, ra);
  x.p = fmaf(s.h6, pp + kp, x.p);
  const float q = fmaf(s.h6q, pq + kq, x.q);
  rl += pl;
  ra += pa;
  ml = fmaf(s.h6, rl, ml);
  ma = fmaf(s.h6, ra, ma);
  quad_mul_inv(C, rl, ra, yl, ya);
  x.v = fmaf(s.third, yl, x.v);
  x.w = fmaf(s.third, ya, x.w);
  if constexpr (LAG) {
    dl *= s.rho;
    da *= s.rho;
  }
  x.q = quad_normalise(q);
}

// M nu
__device__ __forceinline__ void quad_momentum(const QuadMass& M, float v, float w, float& ml,
                                              float& ma) {
  ml = fmaf(qperm<kSwapXY>(w), M.cl, M.l * v);
  // the angular rows of M nu are written M_diag w + (coupling v)
  ma = fmaf(M.a, w, qperm<kSwapXY>(v) * M.ca);
}

// begin_control_step: the command wrench (gl, ga), the lag wrench (dl, da) and
// the lag states at their end-of-control-step value, f_cmd + decay (f - f_cmd);
// SCALED: f_cmd + decay 2^e (f - f_cmd).
template <bool LAG, bool SCALED = false>
__device__ __forceinline__ void quad_command(const QuadThr& t, const float (&act)[2], float decay,
                                             QuadState& x, float& gl, float& ga, float& dl,
                                             float& da, int e = 0) {
  float fcmd[2];
  quad_thrust(t, act, fcmd);
  quad_wrench(t, fcmd, gl, ga);
  dl = da = 0.0f;
  if constexpr (LAG) {
    if (t.lag) {
      const float df[2] = {x.f[0] - fcmd[0], x.f[1] - fcmd[1]};
      quad_wrench(t, df, dl, da);
      x.f[0] = fmaf(decay, SCALED ? ldexpf(df[0], e) : df[0], fcmd[0]);
      x.f[1] = fmaf(decay, SCALED ? ldexpf(df[1], e) : df[1], fcmd[1]);
    }
  }
}

// the same and M nu
template <bool LAG>
__device__ __forceinline__ void quad_begin(const QuadThr& t, const QuadMass& M,
                                           const float (&act)[2], QuadState& x, float& gl,
                                           float& ga, float& dl, float& da, float& ml, float& ma) {
  quad_command<LAG>(t, act, t.rho_s, x, gl, ga, dl, da);
  quad_momentum(M, x.v, x.w, ml, ma);
}

template <bool LAG>
__device__ __forceinline__ void quad_control_step(const QuadLane& L, const QuadConst& C,
                                                  const QuadMass& M, const QuadThr& t,
                                                  const QuadStep& s, const float (&act)[2],
                                                  QuadState& x, int S) {
  float gl, ga, dl, da, ml, ma;
  quad_begin<LAG>(t, M, act, x, gl, ga, dl, da, ml, ma);
  for (int i = 0; i < S; ++i) quad_substep<LAG>(L, C, s, x, ml, ma, gl, ga, dl, da);
}

__device__ __forceinline__ double quad_sum(double x) {
  x += qperm<MG_QP(1, 0, 3, 2)>(x);
  return x + qperm<MG_QP(2, 3, 0, 1)>(x);
}

// A wave's part of the episode statistics, in every quad: lane c takes statistic
// c, the sum of the distances to the targets (lane c's component tg), their
// maximum, the kinetic energy and the count of frozen envs; good: active and not
// frozen.  Quads of a row of 16 lanes by DPP rotations, rows through LDS.
__device__ __forceinline__ double quad_stats(int c, const QuadMass& M, float p, float v, float w,
                                             float tg, bool active, bool good) {
  const double dd = c > 0 ? (double)p - tg : 0.0;
  const double vd = v, wd = w;
  const double al = (double)M.l * vd + (double)M.cl * qperm<kSwapXY>(w);
  const double aa = (double)M.a * wd + (double)M.ca * qperm<kSwapXY>(v);
  const double dist = sqrt(quad_sum(dd * dd));
  const double ke = 0.5 * quad_sum(c > 0 ? vd * al + wd * aa : 0.0);
  double s = c == 3 ? (active && !good ? 1.0 : 0.0) : (good ? (c == 2 ? ke : dist) : 0.0);
  auto join = [&](double o) { s = c == 1 ? fmax(s, o) : s + o; };
  join(qperm<0x124>(s));   // row_ror:4
  join(qperm<0x128>(s));   // row_ror:8
  join(__shfl_xor(s, 16, 64));
  join(__shfl_xor(s, 32, 64));
  return s;
}

// An LDS-only barrier: loads in flight stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

#pragma clang fp contract(fast)

}  // namespace mg
