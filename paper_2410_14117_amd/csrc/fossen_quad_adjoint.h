// fossen_quad_adjoint.h -- the reverse sub-step of fossen_adjoint.h with one env
// spread over a quad of four lanes (fossen_quad.h: lane c holds component c of
// the quaternion and, for c = 1..3, of each 3-vector), for launches too small
// to fill the GPU with one env per lane.  Every value that is read is formed
// by the operations of rhs_core_vjp and rk4_substep_vjp in their order, so
// gradients are bitwise equal up to the sign of zeros.  Lane 0 carries
// don't-care values in the 3-vectors that no other lane reads.
//
// A reverse sub-step is 1700-1850 VALU instructions with one env per lane (the
// chain that a launch of few waves waits for) and about 700 here: a cross
// product is two FMAs for its three components, and each rotated operand is
// one DPP move shared by all the products that read it.
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

// One stage: the state, its rotated components, and the forward intermediates.
struct QuadStage {
  float q, v, w, qw, q1, q2, v1, v2, w1, w2;
  float t, k, a1, a2, b1, b2, el, ea;   // momenta and damping d_L + d_Q |nu|
  float kq, nl, na;                     // TWICE q', nu'
};

__device__ __forceinline__ void quad_stage(const QuadLane& L, const QuadAdjConst& C, float q,
                                           float v, float w, float tl, float ta, QuadStage& s) {
  s.q = q; s.v = v; s.w = w;
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
  s.kq = fmaf(-s.q2, s.w1, fmaf(s.q1, s.w2, q0 * w0));
  s.k = fmaf(qperm<MG_QP(3, 3, 3, 2)>(q), qperm<MG_QP(0, 1, 2, 2)>(q) * L.kf,
             fmaf(qperm<MG_QP(0, 0, 0, 1)>(q), qperm<MG_QP(0, 2, 1, 1)>(q) * L.kc, L.ke));
  const float a = fmaf(qperm<kSwapXY>(w), C.Mcl, C.Ml * v);
  const float b = fmaf(C.Ma, w, qperm<kSwapXY>(v) * C.Mca);
  s.a1 = qperm<kRot1>(a);
  s.a2 = qperm<kRot2>(a);
  s.b1 = qperm<kRot1>(b);
  s.b2 = qperm<kRot2>(b);
  s.el = fmaf(C.dql, fabsf(v), C.dll);
  s.ea = fmaf(C.dqa, fabsf(w), C.dla);
  const float rl = fmaf(-s.el, v, fmaf(C.wmb, s.k, fmaf(-s.w1, s.a2, fmaf(s.w2, s.a1, tl))));
  float ra = fmaf(-s.v1, s.a2, ta);
  ra = fmaf(s.v2, s.a1, ra);
  ra = fmaf(-s.w1, s.b2, ra);
  ra = fmaf(s.w2, s.b1, ra);
  ra = fmaf(qperm<kSwapXY>(s.k), C.hz, ra);
  ra = fmaf(-s.ea, w, ra);
  s.nl = fmaf(qperm<kSwapXY>(ra), C.Icl, C.Il * rl);
  s.na = fmaf(C.Ia, ra, qperm<kSwapXY>(rl) * C.Ica);
}

// rhs_core_vjp: adjoints (xq, xv, xw) of the stage's state and (f, m) of its
// wrench from those of its rates, (gp, gq, gl, ga).
__device__ __forceinline__ void quad_stage_vjp(const QuadAdjLane& L, bool lane0,
                                               const QuadAdjConst& C, const QuadStage& s, float gp,
                                               float gq, float gl, float ga, float& xq, float& xv,
                                               float& xw, float& f, float& m, QuadTheta& th) {
  f = fmaf(qperm<kSwapXY>(ga), C.Icl, C.Il * gl);
  m = fmaf(C.Ia, ga, qperm<kSwapXY>(gl) * C.Ica);
  const float f1 = qperm<kRot1>(f), f2 = qperm<kRot2>(f);
  const float m1 = qperm<kRot1>(m), m2 = qperm<kRot2>(m);
  th.mal = fmaf(-f, s.nl, th.mal);
  th.maa = fmaf(-m, s.na, th.maa);
  th.wmb = fmaf(qbcast<1>(s.k), qbcast<1>(f), th.wmb);
  th.wmb = fmaf(qbcast<2>(s.k), qbcast<2>(f), th.wmb);
  th.wmb = fmaf(qbcast<3>(s.k), qbcast<3>(f), th.wmb);
  th.hz = fmaf(-qbcast<2>(s.k), qbcast<1>(m), th.hz);
  th.hz = fmaf(qbcast<1>(s.k), qbcast<2>(m), th.hz);
  const float ebl = -s.v * f, eba = -s.w * m;
  th.dll += ebl;
  th.dla += eba;
  th.dql = fmaf(ebl, fabsf(s.v), th.dql);
  th.dqa = fmaf(eba, fabsf(s.w), th.dqa);
  const float el = fmaf(C.dql, fabsf(s.v), s.el), ea = fmaf(C.dqa, fabsf(s.w), s.ea);
  const float ab = fmaf(-s.v2, m1, fmaf(s.v1, m2, fmaf(-s.w2, f1, s.w1 * f2)));
  const float bb = fmaf(-s.w2, m1, s.w1 * m2);
  xv = fmaf(-s.a1, m2, fmaf(s.a2, m1, fmaf(-el, f, gp)));
  xw = fmaf(-s.b1, m2, fmaf(s.b2, m1, fmaf(-s.a1, f2, fmaf(s.a2, f1, -ea * m))));
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
  th.mal = fmaf(s.v, ab, th.mal);
  th.maa = fmaf(s.w, bb, th.maa);
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

// Adjoint of the state: lane c's components.
struct QuadLambda {
  float p, q, v, w, f[2];
};

// rk4_substep_vjp: lam holds dL/d(output) on entry, dL/d(input) on exit.
template <bool LAG>
__device__ __forceinline__ void quad_substep_vjp(const QuadLane& L, const QuadAdjLane& LA,
                                                 const QuadAdjConst& C, const QuadThr& thr,
                                                 const QuadThrCols& cols, const QuadStep& k,
                                                 const QuadState& y, const float (&fcmd)[2],
                                                 float gl, float ga, QuadLambda& lam,
                                                 float (&fcb)[2], float& gcl, float& gca,
                                                 QuadTheta& th) {
  const bool lane0 = L.c == 0;
  float dl = 0.0f, da = 0.0f;
  if constexpr (LAG) {
    if (thr.lag) {
      const float df[2] = {y.f[0] - fcmd[0], y.f[1] - fcmd[1]};
      quad_wrench(thr, df, dl, da);
    }
  }
  // the stages and the quaternion before its renormalisation
  auto tl = [&](float sg) { return LAG ? fmaf(sg, dl, gl) : gl; };
  auto ta = [&](float sg) { return LAG ? fmaf(sg, da, ga) : ga; };
  QuadStage s1, s2, s3, s4;
  quad_stage(L, C, y.q, y.v, y.w, LAG ? gl + dl : gl, LAG ? ga + da : ga, s1);
  float acc = s1.kq;
  quad_stage(L, C, fmaf(k.h2q, s1.kq, y.q), fmaf(k.h2, s1.nl, y.v), fmaf(k.h2, s1.na, y.w),
             tl(k.s2), ta(k.s2), s2);
  acc = fmaf(2.0f, s2.kq, acc);
  quad_stage(L, C, fmaf(k.h2q, s2.kq, y.q), fmaf(k.h2, s2.nl, y.v), fmaf(k.h2, s2.na, y.w),
             tl(k.s3), ta(k.s3), s3);
  acc = fmaf(2.0f, s3.kq, acc);
  quad_stage(L, C, fmaf(k.dtq, s3.kq, y.q), fmaf(k.dt, s3.nl, y.v), fmaf(k.dt, s3.na, y.w),
             tl(k.s4), ta(k.s4), s4);
  const float qt = fmaf(k.h6q, acc + s4.kq, y.q);
  const float bw = qbcast<0>(qt), bx = qbcast<1>(qt), by = qbcast<2>(qt), bz = qbcast<3>(qt);
  const float inv = rsqrt_t(fmaf(bz, bz, fmaf(by, by, fmaf(bw, bw, bx * bx))));
  const float qo = qt * inv, dq = qo * lam.q;
  const float dot = ((qbcast<0>(dq) + qbcast<1>(dq)) + qbcast<2>(dq)) + qbcast<3>(dq);
  const float zq = fmaf(-qo, dot, lam.q) * inv;
  // the combination and the stages in reverse
  const float p1 = k.h6 * lam.p, p2 = (2.0f * k.h6) * lam.p;
  const float q1 = k.h6q * zq, q2 = (2.0f * k.h6q) * zq;
  const float v1 = k.h6 * lam.v, v2 = (2.0f * k.h6) * lam.v;
  const float w1 = k.h6 * lam.w, w2 = (2.0f * k.h6) * lam.w;
  float yq = zq, yv = lam.v, yw = lam.w, xq, xv, xw;
  float f1, m1, f2, m2, f3, m3, f4, m4;
  quad_stage_vjp(LA, lane0, C, s4, p1, q1, v1, w1, xq, xv, xw, f4, m4, th);
  yq += xq; yv += xv; yw += xw;
  quad_stage_vjp(LA, lane0, C, s3, p2, fmaf(k.dtq, xq, q2), fmaf(k.dt, xv, v2),
                 fmaf(k.dt, xw, w2), xq, xv, xw, f3, m3, th);
  yq += xq; yv += xv; yw += xw;
  quad_stage_vjp(LA, lane0, C, s2, p2, fmaf(k.h2q, xq, q2), fmaf(k.h2, xv, v2),
                 fmaf(k.h2, xw, w2), xq, xv, xw, f2, m2, th);
  yq += xq; yv += xv; yw += xw;
  quad_stage_vjp(LA, lane0, C, s1, p1, fmaf(k.h2q, xq, q1), fmaf(k.h2, xv, v1),
                 fmaf(k.h2, xw, w1), xq, xv, xw, f1, m1, th);
  lam.q = yq + xq;
  lam.v = yv + xv;
  lam.w = yw + xw;
  gcl += (f1 + f2) + (f3 + f4);
  gca += (m1 + m2) + (m3 + m4);
  if constexpr (LAG) {
    if (thr.lag) {
      const float bl = fmaf(k.s4, f4, fmaf(k.s3, f3, fmaf(k.s2, f2, f1)));
      const float ba = fmaf(k.s4, m4, fmaf(k.s3, m3, fmaf(k.s2, m2, m1)));
      float dfb[2] = {k.rho * lam.f[0], k.rho * lam.f[1]};
      quad_cols_add(cols, bl, ba, dfb);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        fcb[h] += lam.f[h] - dfb[h];
        lam.f[h] = dfb[h];
      }
    }
  }
}

// throttle_vjp of the lane's two throttles
__device__ __forceinline__ void quad_throttle_vjp(const QuadThr& t, const QuadThrCols& cols,
                                                  const float (&a)[2], float (&fcb)[2], float gcl,
                                                  float gca, float (&ab)[2]) {
  quad_cols_add(cols, gcl, gca, fcb);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const bool inside = !(a[h] > 1.0f) && !(a[h] < -1.0f);
    const float slope = t.map ? (2.0f * t.f_max) * fabsf(a[h]) : t.f_max;
    ab[h] = inside ? fcb[h] * slope : 0.0f;
  }
}

#pragma clang fp contract(fast)

}  // namespace mg
