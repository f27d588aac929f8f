// fossen_quad_adjoint.h -- the reverse sub-step of fossen_adjoint.h with one env
// spread over a quad of four lanes (fossen_quad.h: lane c holds component c of
// the quaternion and, for c = 1..3, of each 3-vector), for launches too small
// to fill the GPU with one env per lane.  Every value that is read is formed
// by the operations of rhs_core_vjp and rk4_substep_vjp in their order, so
// gradients are bitwise equal up to the sign of zeros.  Lane 0 carries
// don't-care values in the 3-vectors that no other lane reads.
//
// A reverse sub-step is 1700-1850 VALU instructions with one env per lane (the
// chain that a launch of few waves waits for) and 660-740 here, 345 of them in
// the chain of state adjoints: a cross product is two FMAs for its three
// components, and each rotated operand is one DPP move shared by all the
// products that read it.
#pragma once

#include "fossen_quad.h"

namespace mg {

#pragma clang fp contract(off)

template <int LANE>
__device__ __forceinline__ float qbcast(float x) {
  return qperm<MG_QP(LANE, LANE, LANE, LANE)>(x);
}

// Factors of lane c in the reverse of k = R^T e3.
struct QuadAdjLane {
  float kb;   // x, y, z: 1, -1, 1
  float kc;   // -2, -2, 0
  float ks;   // 1, -1, 0
};
__device__ __forceinline__ QuadAdjLane quad_adj_lane(int c) {
  QuadAdjLane L;
  L.kb = c == 2 ? -1.0f : 1.0f;
  L.kc = c == 3 ? 0.0f : -2.0f;
  L.ks = c == 3 ? 0.0f : L.kb;
  return L;
}

// Per-env constants: M and M^-1 (diagonal and coupling), damping, W - B and
// (-h_z, h_z, 0).
struct QuadAdjConst {
  float Ml, Ma, Mcl, Mca, Il, Ia, Icl, Ica;
  float dll, dla, dql, dqa, wmb, hz;
};
__device__ __forceinline__ void load_quad_adj_const(const float* der, int64_t Ep, uint32_t j4,
                                                    int c, QuadAdjConst& A) {
  QuadConst C;
  QuadMass M;
  load_quad_const(der, Ep, j4, c, 1.0f, C, M);   // factor 1: M^-1 itself
  A.Ml = M.l; A.Ma = M.a; A.Mcl = M.cl; A.Mca = M.ca;
  A.Il = C.Al; A.Ia = C.Aa; A.Icl = C.Acl; A.Ica = C.Aca;
  A.dll = C.dll; A.dla = C.dla; A.dql = C.dql; A.dqa = C.dqa;
  A.wmb = C.wmb; A.hz = C.hz;
}

// Columns c and c + 4 of the allocation matrix (the lane's thrusters).
struct QuadThrCols {
  float b[2][6];
};
__device__ __forceinline__ void load_quad_cols(const ClassConst* cc, int c, QuadThrCols& t) {
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int j = 0; j < 6; ++j) t.b[h][j] = cc->B[j][c + 4 * h];
}

// s[h] += (B^T (l, a)) of the lane's thrusters, rows in order
__device__ __forceinline__ void quad_cols_add(const QuadThrCols& t, float l, float a,
                                              float (&s)[2]) {
  const float r[6] = {qbcast<1>(l), qbcast<2>(l), qbcast<3>(l),
                      qbcast<1>(a), qbcast<2>(a), qbcast<3>(a)};
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int j = 0; j < 6; ++j) s[h] = fmaf(t.b[h][j], r[j], s[h]);
}

// Lane c's rows of the parameter adjoints (wmb and hz the same in every lane).
struct QuadTheta {
  float mal, maa, dll, dla, dql, dqa, wmb, hz;
};

// One stage's forward values, those the chain of state adjoints reads ...
struct QuadStage {
  float q, qw, q1, q2, v1, v2, w, w1, w2;  // state and its rotated components
  float t, a1, a2, b1, b2;                 // 2 q_v x v, momenta
  float el, ea;                            // d_L + 2 d_Q |nu|
};
// ... and those the parameter adjoints read.
struct QuadStageTheta {
  float v, w, k, nl, na;                   // nu' in (nl, na)
};

// kq: TWICE q'
__device__ __forceinline__ void quad_stage(const QuadLane& L, const QuadAdjConst& C, float q,
                                           float v, float w, float tl, float ta, QuadStage& s,
                                           QuadStageTheta& st, float& kq) {
  s.q = q;
  s.w = st.w = w;
  st.v = v;
  const float q0 = qperm<kQW>(q);         // w, lane 0: z
  s.qw = qbcast<0>(q);
  s.q1 = qperm<kQRot1>(q);
  s.q2 = qperm<kQRot2>(q);
  s.v1 = qperm<kRot1>(v);
  s.v2 = qperm<kRot2>(v);
  s.w1 = qperm<kRot1>(w);
  const float w0 = qperm<MG_QP(3, 1, 2, 3)>(w) * L.sg;
  s.w2 = qperm<kRot2>(w) * L.sg;          // lane 0 negated, as quad_residual
  const float th = fmaf(s.q1, s.v2, -(s.q2 * s.v1));
  s.t = th + th;
  kq = fmaf(-s.q2, s.w1, fmaf(s.q1, s.w2, q0 * w0));
  st.k = fmaf(qperm<MG_QP(3, 3, 3, 2)>(q), qperm<MG_QP(0, 1, 2, 2)>(q) * L.kf,
             fmaf(qperm<MG_QP(0, 0, 0, 1)>(q), qperm<MG_QP(0, 2, 1, 1)>(q) * L.kc, L.ke));
  const float a = fmaf(qperm<kSwapXY>(w), C.Mcl, C.Ml * v);
  const float b = fmaf(C.Ma, w, qperm<kSwapXY>(v) * C.Mca);
  s.a1 = qperm<kRot1>(a);
  s.a2 = qperm<kRot2>(a);
  s.b1 = qperm<kRot1>(b);
  s.b2 = qperm<kRot2>(b);
  const float el = fmaf(C.dql, fabsf(v), C.dll), ea = fmaf(C.dqa, fabsf(w), C.dla);
  const float rl = fmaf(-el, v, fmaf(C.wmb, st.k, fmaf(-s.w1, s.a2, fmaf(s.w2, s.a1, tl))));
  float ra = fmaf(-s.v1, s.a2, ta);
  ra = fmaf(s.v2, s.a1, ra);
  ra = fmaf(-s.w1, s.b2, ra);
  ra = fmaf(s.w2, s.b1, ra);
  ra = fmaf(qperm<kSwapXY>(st.k), C.hz, ra);
  ra = fmaf(-ea, w, ra);
  st.nl = fmaf(qperm<kSwapXY>(ra), C.Icl, C.Il * rl);
  st.na = fmaf(C.Ia, ra, qperm<kSwapXY>(rl) * C.Ica);
  s.el = fmaf(C.dql, fabsf(v), el);
  s.ea = fmaf(C.dqa, fabsf(w), ea);
}

// A sub-step's four stages and its quaternion's renormalisation: q = qo = qt inv.
struct QuadStages {
  QuadStage s[4];
  QuadStageTheta t[4];
  float qo, inv;
};
template <bool LAG>
__device__ __forceinline__ void quad_stages(const QuadLane& L, const QuadAdjConst& C,
                                            const QuadThr& thr, const QuadStep& k,
                                            const QuadState& y, const float (&fcmd)[2], float gl,
                                            float ga, QuadStages& o) {
  float dl = 0.0f, da = 0.0f;
  if constexpr (LAG) {
    if (thr.lag) {
      const float df[2] = {y.f[0] - fcmd[0], y.f[1] - fcmd[1]};
      quad_wrench(thr, df, dl, da);
    }
  }
  auto tl = [&](float sg) { return LAG ? fmaf(sg, dl, gl) : gl; };
  auto ta = [&](float sg) { return LAG ? fmaf(sg, da, ga) : ga; };
  float kq;
  quad_stage(L, C, y.q, y.v, y.w, LAG ? gl + dl : gl, LAG ? ga + da : ga, o.s[0], o.t[0], kq);
  float acc = kq;
  quad_stage(L, C, fmaf(k.h2q, kq, y.q), fmaf(k.h2, o.t[0].nl, y.v), fmaf(k.h2, o.t[0].na, y.w),
             tl(k.s2), ta(k.s2), o.s[1], o.t[1], kq);
  acc = fmaf(2.0f, kq, acc);
  quad_stage(L, C, fmaf(k.h2q, kq, y.q), fmaf(k.h2, o.t[1].nl, y.v), fmaf(k.h2, o.t[1].na, y.w),
             tl(k.s3), ta(k.s3), o.s[2], o.t[2], kq);
  acc = fmaf(2.0f, kq, acc);
  quad_stage(L, C, fmaf(k.dtq, kq, y.q), fmaf(k.dt, o.t[2].nl, y.v), fmaf(k.dt, o.t[2].na, y.w),
             tl(k.s4), ta(k.s4), o.s[3], o.t[3], kq);
  const float qt = fmaf(k.h6q, acc + kq, y.q);
  const float bw = qbcast<0>(qt), bx = qbcast<1>(qt), by = qbcast<2>(qt), bz = qbcast<3>(qt);
  o.inv = rsqrt_t(fmaf(bz, bz, fmaf(by, by, fmaf(bw, bw, bx * bx))));
  o.qo = qt * o.inv;
}

// What the parameter and thruster adjoints read of a stage's reverse: the
// adjoint of its wrench (f, m) and of its momenta (ab, bb).
struct QuadStageOut {
  float f, m, ab, bb;
};

// rhs_core_vjp without the parameters: adjoints (xq, xv, xw) of the stage's state
// from those of its rates, (gp, gq, gl, ga).
__device__ __forceinline__ void quad_stage_vjp(const QuadAdjLane& L, bool lane0,
                                               const QuadAdjConst& C, const QuadStage& s, float gp,
                                               float gq, float gl, float ga, float& xq, float& xv,
                                               float& xw, QuadStageOut& o) {
  const float f = fmaf(qperm<kSwapXY>(ga), C.Icl, C.Il * gl);
  const float m = fmaf(C.Ia, ga, qperm<kSwapXY>(gl) * C.Ica);
  const float f1 = qperm<kRot1>(f), f2 = qperm<kRot2>(f);
  const float m1 = qperm<kRot1>(m), m2 = qperm<kRot2>(m);
  const float ab = fmaf(-s.v2, m1, fmaf(s.v1, m2, fmaf(-s.w2, f1, s.w1 * f2)));
  const float bb = fmaf(-s.w2, m1, s.w1 * m2);
  o = {f, m, ab, bb};
  xv = fmaf(-s.a1, m2, fmaf(s.a2, m1, fmaf(-s.el, f, gp)));
  xw = fmaf(-s.b1, m2, fmaf(s.b2, m1, fmaf(-s.a1, f2, fmaf(s.a2, f1, -s.ea * m))));
  const float gw = qbcast<0>(gq), gv1 = qperm<kQRot1>(gq), gv2 = qperm<kQRot2>(gq);
  const float gp1 = qperm<kRot1>(gp), gp2 = qperm<kRot2>(gp);
  xw = fmaf(-gv2, s.q1, fmaf(gv1, s.q2, fmaf(s.qw, gq, fmaf(-s.q, gw, xw))));
  const float tb = fmaf(-gp2, s.q1, fmaf(gp1, s.q2, s.qw * gp));
  const float tb2 = tb + tb;
  const float kb = fmaf(-qperm<kSwapXY>(m), C.hz, C.wmb * f);
  const float kb2 = kb + kb;
  float qb = fmaf(-s.w2, gv1, fmaf(s.w1, gv2, -s.w * gw));
  qb = fmaf(-qperm<kRot2>(s.t), gp1, fmaf(qperm<kRot1>(s.t), gp2, qb));
  float d = fmaf(s.t, gp, s.w * gq);
  xv = fmaf(C.Mcl, qperm<kSwapXY>(bb), fmaf(C.Ml, ab, xv));
  xw = fmaf(C.Mca, qperm<kSwapXY>(ab), fmaf(C.Ma, bb, xw));
  const float t1 = qperm<kRot1>(tb2), t2 = qperm<kRot2>(tb2);
  xv = fmaf(-t2, s.q1, fmaf(t1, s.q2, xv));
  qb = fmaf(-s.v2, t1, fmaf(s.v1, t2, qb));
  // k = R^T e3: x (qz kx + qw ky - 2 qx kz), y (qz ky - qw kx - 2 qy kz), z (qx kx + qy ky)
  qb = fmaf(qperm<MG_QP(0, 3, 3, 1)>(s.q), qperm<MG_QP(0, 1, 2, 1)>(kb2), qb);
  qb = fmaf(qperm<MG_QP(0, 0, 0, 2)>(s.q) * L.kb, qperm<MG_QP(0, 2, 1, 2)>(kb2), qb);
  qb = fmaf(s.q * L.kc, qbcast<3>(kb2), qb);
  d = fmaf(s.q * L.ks, qperm<kSwapXY>(kb2), d);
  const float dw = (qbcast<1>(d) + qbcast<2>(d)) + qbcast<3>(d);
  xq = lane0 ? dw : qb;
}

// The parameters' part of rhs_core_vjp.
__device__ __forceinline__ void quad_stage_theta(const QuadStageTheta& s, const QuadStageOut& o,
                                                 QuadTheta& th) {
  th.mal = fmaf(-o.f, s.nl, th.mal);
  th.maa = fmaf(-o.m, s.na, th.maa);
  th.wmb = fmaf(qbcast<1>(s.k), qbcast<1>(o.f), th.wmb);
  th.wmb = fmaf(qbcast<2>(s.k), qbcast<2>(o.f), th.wmb);
  th.wmb = fmaf(qbcast<3>(s.k), qbcast<3>(o.f), th.wmb);
  th.hz = fmaf(-qbcast<2>(s.k), qbcast<1>(o.m), th.hz);
  th.hz = fmaf(qbcast<1>(s.k), qbcast<2>(o.m), th.hz);
  const float ebl = -s.v * o.f, eba = -s.w * o.m;
  th.dll += ebl;
  th.dla += eba;
  th.dql = fmaf(ebl, fabsf(s.v), th.dql);
  th.dqa = fmaf(eba, fabsf(s.w), th.dqa);
  th.mal = fmaf(s.v, o.ab, th.mal);
  th.maa = fmaf(s.w, o.bb, th.maa);
}

// Adjoint of the rigid-body state: lane c's components.
struct QuadLambda {
  float p, q, v, w;
};

// rk4_substep_vjp's chain of state adjoints: lam holds dL/d(output) on entry,
// dL/d(input) on exit; stage(i, s) gives stage i's forward values, out(i, o)
// takes what its reverse leaves for the parameters; stages 3, 2, 1, 0.
template <class STAGE, class OUT>
__device__ __forceinline__ void quad_substep_vjp(int c, const QuadAdjLane& LA,
                                                 const QuadAdjConst& C, const QuadStep& k,
                                                 float qo, float inv, STAGE stage, OUT out,
                                                 QuadLambda& lam) {
  const bool lane0 = c == 0;
  const float dq = qo * lam.q;
  const float dot = ((qbcast<0>(dq) + qbcast<1>(dq)) + qbcast<2>(dq)) + qbcast<3>(dq);
  const float zq = fmaf(-qo, dot, lam.q) * inv;
  // the combination and the stages in reverse
  const float p1 = k.h6 * lam.p, p2 = (2.0f * k.h6) * lam.p;
  const float q1 = k.h6q * zq, q2 = (2.0f * k.h6q) * zq;
  const float v1 = k.h6 * lam.v, v2 = (2.0f * k.h6) * lam.v;
  const float w1 = k.h6 * lam.w, w2 = (2.0f * k.h6) * lam.w;
  float yq = zq, yv = lam.v, yw = lam.w, xq, xv, xw;
  QuadStageOut o;
  quad_stage_vjp(LA, lane0, C, stage(3), p1, q1, v1, w1, xq, xv, xw, o);
  out(3, o);
  yq += xq; yv += xv; yw += xw;
  quad_stage_vjp(LA, lane0, C, stage(2), p2, fmaf(k.dtq, xq, q2), fmaf(k.dt, xv, v2),
                 fmaf(k.dt, xw, w2), xq, xv, xw, o);
  out(2, o);
  yq += xq; yv += xv; yw += xw;
  quad_stage_vjp(LA, lane0, C, stage(1), p2, fmaf(k.h2q, xq, q2), fmaf(k.h2, xv, v2),
                 fmaf(k.h2, xw, w2), xq, xv, xw, o);
  out(1, o);
  yq += xq; yv += xv; yw += xw;
  quad_stage_vjp(LA, lane0, C, stage(0), p1, fmaf(k.h2q, xq, q1), fmaf(k.h2, xv, v1),
                 fmaf(k.h2, xw, w1), xq, xv, xw, o);
  out(0, o);
  lam.q = yq + xq;
  lam.v = yv + xv;
  lam.w = yw + xw;
}

// Adjoints of the lane's two thrusters: of their states, of the commanded
// thrust, and of the command's wrench.
struct QuadThrBar {
  float lam[2], fcb[2], gcl, gca;
};

// rk4_substep_vjp's thrusters, from the stages' wrench adjoints.
template <bool LAG>
__device__ __forceinline__ void quad_thrusters_vjp(const QuadThr& thr, const QuadThrCols& cols,
                                                   const QuadStep& k, const QuadStageOut (&o)[4],
                                                   QuadThrBar& b) {
  b.gcl += (o[0].f + o[1].f) + (o[2].f + o[3].f);
  b.gca += (o[0].m + o[1].m) + (o[2].m + o[3].m);
  if constexpr (LAG) {
    if (thr.lag) {
      const float bl = fmaf(k.s4, o[3].f, fmaf(k.s3, o[2].f, fmaf(k.s2, o[1].f, o[0].f)));
      const float ba = fmaf(k.s4, o[3].m, fmaf(k.s3, o[2].m, fmaf(k.s2, o[1].m, o[0].m)));
      float dfb[2] = {k.rho * b.lam[0], k.rho * b.lam[1]};
      quad_cols_add(cols, bl, ba, dfb);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        b.fcb[h] += b.lam[h] - dfb[h];
        b.lam[h] = dfb[h];
      }
    }
  }
}

// throttle_vjp of the lane's two throttles
__device__ __forceinline__ void quad_throttle_vjp(const QuadThr& t, const QuadThrCols& cols,
                                                  const float (&a)[2], QuadThrBar& b,
                                                  float (&ab)[2]) {
  quad_cols_add(cols, b.gcl, b.gca, b.fcb);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const bool inside = !(a[h] > 1.0f) && !(a[h] < -1.0f);
    const float slope = t.map ? (2.0f * t.f_max) * fabsf(a[h]) : t.f_max;
    ab[h] = inside ? b.fcb[h] * slope : 0.0f;
  }
}

#pragma clang fp contract(fast)

}  // namespace mg
