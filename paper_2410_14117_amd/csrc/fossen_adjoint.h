// fossen_adjoint.h -- reverse mode of the RK4 sub-step of fossen_device.h:
// vector-Jacobian products of the right-hand side and of one whole sub-step
// (stages, combination, quaternion renormalisation, closed-form lag stages),
// with respect to the state, the commanded thrust and the per-env
// hydrodynamic parameters theta = (M_A(6), D_L(6), D_Q(6), B).
//
// Everything is exact for the discrete map the forward kernels compute; the
// forward intermediates are recomputed from the sub-step input.
#pragma once

#include "fossen_device.h"

namespace mg {

// Adjoints of the parameter-dependent constants: diagonal of M (M_A enters
// there; the off-diagonal m z_g terms do not depend on theta), the damping
// diagonals, W - B and h_z = W z_g - B z_b.
template <class T>
struct ThetaBar {
  T ma[6], dl[6], dq[6], wmb, hz;
};

template <class T>
__host__ __device__ __forceinline__ void theta_bar_zero(ThetaBar<T>& t) {
#pragma unroll
  for (int i = 0; i < 6; ++i) t.ma[i] = t.dl[i] = t.dq[i] = T(0);
  t.wmb = t.hz = T(0);
}

// The same adjoints held in LDS, [20][kBlock] floats (slot k of a lane at
// col + k kBlock), for the two-wave trajectory-reading sweep, which has 256
// registers and would otherwise spill inside the sub-step VJP: each
// += / -= is a load, the same operation and a store, so the sums are those of
// ThetaBar, bitwise.  theta_bar_fence, a compiler-only memory barrier placed
// between the stage VJPs, keeps the compiler from holding the slots in
// registers across them (which would bring the register pressure back); for
// ThetaBar (registers) it is a no-op.
struct LdsAcc {
  float* p;
  __device__ __forceinline__ void operator+=(float v) const { *p = *p + v; }
  __device__ __forceinline__ void operator-=(float v) const { *p = *p - v; }
};
struct LdsAccRow {
  float* p;
  __device__ __forceinline__ LdsAcc operator[](int i) const { return {p + i * kBlock}; }
};
struct ThetaBarLds {
  LdsAccRow ma, dl, dq;
  LdsAcc wmb, hz;
};
// slot k of a lane's column: ma 0-5, dl 6-11, dq 12-17, wmb 18, hz 19
__device__ __forceinline__ ThetaBarLds theta_bar_lds(float* col) {
#pragma unroll
  for (int k = 0; k < 20; ++k) col[k * kBlock] = 0.0f;
  return {{col}, {col + 6 * kBlock}, {col + 12 * kBlock}, {col + 18 * kBlock},
          {col + 19 * kBlock}};
}
template <class T>
__host__ __device__ __forceinline__ void theta_bar_fence(ThetaBar<T>&) {}
__device__ __forceinline__ void theta_bar_fence(ThetaBarLds&) { asm volatile("" ::: "memory"); }
template <class T>
__host__ __device__ __forceinline__ T theta_bar_get(const ThetaBar<T>& t, int k) {
  return k < 6 ? t.ma[k] : k < 12 ? t.dl[k - 6] : k < 18 ? t.dq[k - 12] : k == 18 ? t.wmb : t.hz;
}
__device__ __forceinline__ float theta_bar_get(const ThetaBarLds& t, int k) {
  return *(volatile float*)(t.ma.p + k * kBlock);
}

// Nothing is scheduled across it: the stage VJPs, which hold the most values of a
// sub-step, each begin where the one before has ended.  Without it the compiler
// interleaves them (one wave per SIMD, 20 000 lag-free Heavies, 8 control steps of 4
// sub-steps: backward 113 against 106 us) and, in the two-wave sweeps, spills for it.
__host__ __device__ __forceinline__ void sched_fence() {
#ifdef __HIP_DEVICE_COMPILE__
  __builtin_amdgcn_sched_barrier(0);
#endif
}

// A factor the compiler takes for another value than it has been: products with it
// are formed again instead of being kept.
template <class T>
__host__ __device__ __forceinline__ T formed_again(T v) {
#ifdef __HIP_DEVICE_COMPILE__
  asm volatile("" : "+s"(v));
#endif
  return v;
}

// dL/d(x, tau, theta) of xd = rhs_core(x, tau) given xdb = dL/dxd.
// Writes xb (rows 3..12; the position rows receive nothing) and taub and
// accumulates into thb.
//
// Written on 3-vectors, component i with i1 = i + 1 and i2 = i + 2 (mod 3) and
// every FMA explicit: the same formulas in the same order serve the kernels
// that hold one component per lane (fossen_quad_adjoint.h), bit for bit.  With
// t = 2 q_v x v, k = R^T e3, [a; b] = M nu and [f; m] = M^-1 (g_v, g_w) for the
// rates' adjoints (g_p, g_q, g_v, g_w):
//   a' = w x f + v x m,  b' = w x m,  k' = (W-B) f + (h_z m_y, -h_z m_x, 0)
//   v' = g_p - E_l f - a x m + (M (a', b'))_l + 2 t' x q_v
//   w' = -E_a m - a x f - b x m + (M (a', b'))_a - q_v g_q0 + q_w g_qv + g_qv x q_v
//   t' = q_w g_p + g_p x q_v,  E = d_L + 2 d_Q |nu|
//   q_v' = -w g_q0 + w x g_qv + t x g_p + 2 v x t' + (rows of k)
//   q_w' = w . g_qv + t . g_p + 2 (q_x k'_y - q_y k'_x)
//
// TIGHT (the two-wave recomputing sweeps, which spill): its parts in turn, in an
// order that ends each value's life early.  With the wrenches formed again (below),
// 150 000 lagged Heavies, 8 control steps of 2 sub-steps, 304 -> 238 us recomputed
// first and 288 -> 285 us segment by segment; without a lag 189 -> 184 and 198 -> 194.
template <bool TIGHT = false, class T, class TB>
__host__ __device__ __forceinline__ void rhs_core_vjp(const T* x, const EnvConstT<T>& P,
                                                      const T (&tau)[6], const T* xdb, T* xb,
                                                      T (&taub)[6], TB& thb) {
  // forward intermediates, as rhs_residual forms them
  const T qw = x[3];
  const T* q = x + 4;
  const T* v = x + 7;
  const T* w = x + 10;
  T xd[7], res[6], mom[6];
  momentum(P, v, mom);
  rhs_residual_m(x, mom, xd, res, P, tau);
  const T* a = mom;
  const T* b = mom + 3;
  const T x2 = q[0] + q[0], y2 = q[1] + q[1], z2 = q[2] + q[2];
  const T t[3] = {fma_t(y2, v[2], -z2 * v[1]), fma_t(z2, v[0], -x2 * v[2]),
                  fma_t(x2, v[1], -y2 * v[0])};
  const T k[3] = {fma_t(x2, q[2], -y2 * qw), fma_t(y2, q[2], x2 * qw),
                  fma_t(-y2, q[1], fma_t(-x2, q[0], T(1)))};
  const T nud[6] = {fma_t(P.Iuq, res[4], P.Iuu * res[0]), fma_t(P.Ivp, res[3], P.Ivv * res[1]),
                    P.Iww * res[2], fma_t(P.Ipp, res[3], P.Ivp * res[1]),
                    fma_t(P.Iqq, res[4], P.Iuq * res[0]), P.Irr * res[5]};

  // nu' = M^-1 r:  rb = M^-1 nudb (M symmetric);  dM_ii gets -rb_i nud_i
  const T* gp = xdb;
  const T gw = xdb[3];
  const T* gv = xdb + 4;
  const T* gn = xdb + 7;
  T rb[6];
  rb[0] = fma_t(P.Iuq, gn[4], P.Iuu * gn[0]);
  rb[1] = fma_t(P.Ivp, gn[3], P.Ivv * gn[1]);
  rb[2] = mul_nc(P.Iww, gn[2]);
  rb[3] = fma_t(P.Ipp, gn[3], P.Ivp * gn[1]);
  rb[4] = fma_t(P.Iqq, gn[4], P.Iuq * gn[0]);
  rb[5] = mul_nc(P.Irr, gn[5]);
  const T* f = rb;
  const T* m = rb + 3;
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    thb.ma[i] -= rb[i] * nud[i];
    taub[i] = rb[i];
  }
  thb.wmb += k[0] * f[0];
  thb.wmb += k[1] * f[1];
  thb.wmb += k[2] * f[2];
  thb.hz -= k[1] * m[0];
  thb.hz += k[0] * m[1];
  T ab[3], bb[3], tb2[3], kb2[3], vb[3], wb[3], qb[3], s[3];
  if constexpr (TIGHT) sched_fence();
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int i1 = (i + 1) % 3, i2 = (i + 2) % 3;
    // damping: e = d_L + d_Q |nu| (d|x|/dx taken as +1 at 0)
    const T ebl = mul_nc(-v[i], f[i]), eba = mul_nc(-w[i], m[i]);
    thb.dl[i] += ebl;
    thb.dl[3 + i] += eba;
    thb.dq[i] += ebl * abs_t(v[i]);
    thb.dq[3 + i] += eba * abs_t(w[i]);
    const T el = fma_t(P.dq[i], abs_t(v[i]), fma_t(P.dq[i], abs_t(v[i]), P.dl[i]));
    const T ea = fma_t(P.dq[3 + i], abs_t(w[i]), fma_t(P.dq[3 + i], abs_t(w[i]), P.dl[3 + i]));
    vb[i] = fma_t(-a[i1], m[i2], fma_t(a[i2], m[i1], fma_t(-el, f[i], gp[i])));
    wb[i] = fma_t(-b[i1], m[i2], fma_t(b[i2], m[i1],
            fma_t(-a[i1], f[i2], fma_t(a[i2], f[i1], mul_nc(-ea, m[i])))));
  }
  if constexpr (TIGHT) sched_fence();
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int i1 = (i + 1) % 3, i2 = (i + 2) % 3;
    // quaternion rows (xd[3..6] = q (x) (0, w)), [a; b] = M nu, k = R^T e3
    wb[i] = fma_t(-gv[i2], q[i1], fma_t(gv[i1], q[i2], fma_t(qw, gv[i], fma_t(-q[i], gw, wb[i]))));
    ab[i] = fma_t(-v[i2], m[i1], fma_t(v[i1], m[i2], fma_t(-w[i2], f[i1], mul_nc(w[i1], f[i2]))));
    bb[i] = fma_t(-w[i2], m[i1], mul_nc(w[i1], m[i2]));
    thb.ma[i] += v[i] * ab[i];
    thb.ma[3 + i] += w[i] * bb[i];
    const T kb = mul_nc(P.wmb, f[i]);
    const T kbi = i == 0 ? fma_t(P.hz, m[1], kb) : (i == 1 ? fma_t(-P.hz, m[0], kb) : kb);
    kb2[i] = kbi + kbi;
  }
  if constexpr (TIGHT) sched_fence();
  vb[0] = fma_t(P.Muq, bb[1], fma_t(P.Muu, ab[0], vb[0]));
  vb[1] = fma_t(P.Mvp, bb[0], fma_t(P.Mvv, ab[1], vb[1]));
  vb[2] = fma_t(P.Mww, ab[2], vb[2]);
  wb[0] = fma_t(P.Mvp, ab[1], fma_t(P.Mpp, bb[0], wb[0]));
  wb[1] = fma_t(P.Muq, ab[0], fma_t(P.Mqq, bb[1], wb[1]));
  wb[2] = fma_t(P.Mrr, bb[2], wb[2]);
  if constexpr (TIGHT) sched_fence();
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int i1 = (i + 1) % 3, i2 = (i + 2) % 3;
    const T tb = fma_t(-gp[i2], q[i1], fma_t(gp[i1], q[i2], mul_nc(qw, gp[i])));
    tb2[i] = tb + tb;
    qb[i] = fma_t(-w[i2], gv[i1], fma_t(w[i1], gv[i2], mul_nc(-w[i], gw)));
    qb[i] = fma_t(-t[i2], gp[i1], fma_t(t[i1], gp[i2], qb[i]));
    s[i] = fma_t(t[i], gp[i], mul_nc(w[i], gv[i]));
  }
  if constexpr (TIGHT) sched_fence();
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int i1 = (i + 1) % 3, i2 = (i + 2) % 3;
    vb[i] = fma_t(-tb2[i2], q[i1], fma_t(tb2[i1], q[i2], vb[i]));
    qb[i] = fma_t(-v[i2], tb2[i1], fma_t(v[i1], tb2[i2], qb[i]));
  }
  // k = R^T e3
  qb[0] = fma_t(-x2, kb2[2], fma_t(qw, kb2[1], fma_t(q[2], kb2[0], qb[0])));
  qb[1] = fma_t(-y2, kb2[2], fma_t(-qw, kb2[0], fma_t(q[2], kb2[1], qb[1])));
  qb[2] = fma_t(q[1], kb2[1], fma_t(q[0], kb2[0], qb[2]));
  s[0] = fma_t(q[0], kb2[1], s[0]);
  s[1] = fma_t(-q[1], kb2[0], s[1]);
  xb[3] = (s[0] + s[1]) + s[2];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    xb[4 + i] = qb[i];
    xb[7 + i] = vb[i];
    xb[10 + i] = wb[i];
  }
}

// Reverse of rk4_substep: y is the sub-step input (D rows), lam holds dL/d(output)
// on entry and dL/dy on exit; dL/d f_cmd and dL/d (B f_cmd) accumulate into fcb and
// gcb, parameter adjoints into thb.  TIGHT: the stage wrenches are formed again
// for the stage VJPs, so that neither they nor the residuals with them are held from
// the forward recomputation on (130 more VALU instructions, 9-22 fewer spilled
// registers).
template <int N, bool LAG, bool TIGHT = false, class T, class TB>
__host__ __device__ __forceinline__ void rk4_substep_vjp(const T* y, const EnvConstT<T>& P,
                                                         const ClassConst& cc,
                                                         const T (&fcmd)[N], const T (&gcmd)[6],
                                                         T dt, T* lam, T (&fcb)[N], T (&gcb)[6],
                                                         TB& thb) {
  const T h2 = T(0.5) * dt, h6 = dt * (T(1) / T(6));
  auto fac = [](int i, T f) { return (i >= 3 && i < 7) ? T(0.5) * f : f; };
  T df[N], dg[6], tau1[6], tau2[6], tau3[6], tau4[6];
  if constexpr (LAG) {
#pragma unroll
    for (int i = 0; i < N; ++i) df[i] = y[13 + i] - fcmd[i];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      T s = mul_nc(T(cc.B[k][0]), df[0]);
#pragma unroll
      for (int i = 1; i < N; ++i) s = fma_t(T(cc.B[k][i]), df[i], s);
      dg[k] = s;
      tau1[k] = gcmd[k] + s;
      tau2[k] = fma_t(T(cc.sigma2), s, gcmd[k]);
      tau3[k] = fma_t(T(cc.sigma3), s, gcmd[k]);
      tau4[k] = fma_t(T(cc.sigma4), s, gcmd[k]);
    }
  } else {
#pragma unroll
    for (int k = 0; k < 6; ++k) tau1[k] = tau2[k] = tau3[k] = tau4[k] = gcmd[k];
  }
  // forward recomputation of the stage inputs and of the pre-normalisation quaternion
  T k[13], acc[13], X2[13], X3[13], X4[13];
  rhs_core(y, k, P, tau1);
#pragma unroll
  for (int i = 0; i < 13; ++i) {
    acc[i] = k[i];
    X2[i] = fma_t(fac(i, h2), k[i], y[i]);
  }
  rhs_core(X2, k, P, tau2);
#pragma unroll
  for (int i = 0; i < 13; ++i) {
    acc[i] = fma_t(T(2), k[i], acc[i]);
    X3[i] = fma_t(fac(i, h2), k[i], y[i]);
  }
  rhs_core(X3, k, P, tau3);
#pragma unroll
  for (int i = 0; i < 13; ++i) {
    acc[i] = fma_t(T(2), k[i], acc[i]);
    X4[i] = fma_t(fac(i, dt), k[i], y[i]);
  }
  rhs_core(X4, k, P, tau4);
  T qt[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) qt[i] = fma_t(fac(3 + i, h6), acc[3 + i] + k[3 + i], y[3 + i]);

  // renormalisation q = qt / |qt|:  dqt = (lam_q - q (q . lam_q)) / |qt|
  const T n2 = fma_t(qt[3], qt[3], fma_t(qt[2], qt[2], fma_t(qt[0], qt[0], qt[1] * qt[1])));
  const T inv = rsqrt_t(n2);
  T qo[4], d[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    qo[i] = qt[i] * inv;
    d[i] = mul_nc(qo[i], lam[3 + i]);
  }
  const T dot = ((d[0] + d[1]) + d[2]) + d[3];
  T zb[13];
#pragma unroll
  for (int i = 0; i < 13; ++i) zb[i] = lam[i];
#pragma unroll
  for (int i = 0; i < 4; ++i) zb[3 + i] = mul_nc(lam[3 + i] - qo[i] * dot, inv);

  // combination z' = y + fac(h6) (k1 + 2 k2 + 2 k3 + k4), then the stages in
  // reverse; the position rows of Xb stay zero
  T yb[13], kb[13], Xb[13], tb1[6], tb2[6], tb3[6], tb4[6];
  auto begin_stage = [&](T sigma, T (&tau)[6]) {
    if constexpr (LAG && TIGHT) {
      const T sg = formed_again(sigma);
#pragma unroll
      for (int j = 0; j < 6; ++j) tau[j] = fma_t(sg, dg[j], gcmd[j]);
    }
    theta_bar_fence(thb);
    sched_fence();
  };
  auto scale = [&](T weight) {   // kb = weight fac(h6) zb
#pragma unroll
    for (int i = 0; i < 13; ++i) kb[i] = mul_nc(weight * fac(i, h6), zb[i]);
  };
  auto add_stage = [&](T c) {    // X = y + fac(c) k: into yb and kb
#pragma unroll
    for (int i = 3; i < 13; ++i) {
      yb[i] += Xb[i];
      kb[i] = fma_t(fac(i, c), Xb[i], kb[i]);
    }
  };
#pragma unroll
  for (int i = 0; i < 13; ++i) yb[i] = zb[i];
  scale(T(1));
  begin_stage(T(cc.sigma4), tau4);
  rhs_core_vjp<TIGHT>(X4, P, tau4, kb, Xb, tb4, thb);   // X4 = y + fac(dt) k3
  scale(T(2));
  add_stage(dt);
  begin_stage(T(cc.sigma3), tau3);
  rhs_core_vjp<TIGHT>(X3, P, tau3, kb, Xb, tb3, thb);   // X3 = y + fac(h2) k2
  scale(T(2));
  add_stage(h2);
  begin_stage(T(cc.sigma2), tau2);
  rhs_core_vjp<TIGHT>(X2, P, tau2, kb, Xb, tb2, thb);   // X2 = y + fac(h2) k1
  scale(T(1));
  add_stage(h2);
  begin_stage(T(1), tau1);
  rhs_core_vjp<TIGHT>(y, P, tau1, kb, Xb, tb1, thb);    // X1 = y
#pragma unroll
  for (int i = 0; i < 3; ++i) lam[i] = yb[i];
#pragma unroll
  for (int i = 3; i < 13; ++i) lam[i] = yb[i] + Xb[i];

  // stage wrenches tau_i = B f_cmd + sigma_i B (f - f_cmd) and f' = f_cmd + rho (f - f_cmd)
  if constexpr (LAG) {
    T dgb[6];
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      gcb[j] += (tb1[j] + tb2[j]) + (tb3[j] + tb4[j]);
      dgb[j] = tb1[j] + T(cc.sigma2) * tb2[j] + T(cc.sigma3) * tb3[j] + T(cc.sigma4) * tb4[j];
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const T fob = lam[13 + i];
      T dfb = T(cc.rho) * fob;
#pragma unroll
      for (int j = 0; j < 6; ++j) dfb = fma_t(T(cc.B[j][i]), dgb[j], dfb);
      fcb[i] += fob - dfb;
      lam[13 + i] = dfb;
    }
    (void)dg;
  } else {
#pragma unroll
    for (int j = 0; j < 6; ++j) gcb[j] += (tb1[j] + tb2[j]) + (tb3[j] + tb4[j]);
  }
}

// dL/d throttle from dL/d f_cmd (and dL/d (B f_cmd)), through the clamp and the thrust map.
template <int N, class T>
__host__ __device__ __forceinline__ void throttle_vjp(const ClassConst& cc, const T (&a)[N],
                                                      T (&fcb)[N], const T (&gcb)[6],
                                                      T (&ab)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    T s = fcb[i];
#pragma unroll
    for (int j = 0; j < 6; ++j) s = fma_t(T(cc.B[j][i]), gcb[j], s);
    const bool inside = !(a[i] > T(1)) && !(a[i] < T(-1));
    const T slope = cc.thr_map ? T(2) * T(cc.f_max) * abs_t(a[i]) : T(cc.f_max);
    ab[i] = inside ? s * slope : T(0);
  }
}

// ---- the backward of one env over a checkpointed rollout -------------------
// (kernels_adjoint.hip launches these, one lane per env; host and device code,
// so that the same source also runs on the CPU in tests)

template <int N>
__host__ __device__ __forceinline__ void load_command(const ClassConst& cc, const AdjArgs& a, int t,
                                             int64_t c, float (&act)[N], float (&fcmd)[N],
                                             float (&gcmd)[6]) {
  const float* af = a.actions + (int64_t)t * a.n_max * a.E + c;
#pragma unroll
  for (int i = 0; i < N; ++i) act[i] = af[i * a.E];
  thrust_command<N>(cc, act, fcmd);
  command_wrench<N>(cc, fcmd, gcmd);
}

// Recomputes the sub-step inputs of control steps [t0, t1) from the state x
// at t0 into segbuf rows (t - base) * S + s.  The forward sets the lag states
// to their end-of-control-step value at the start; the sub-step inputs the VJP
// linearises about carry the lag states of each sub-step, f_cmd + rho^s
// (f - f_cmd), kept here in fs.
// Used by k_adj_recompute only: the backward keeps its own copy of this loop
// (see adj_bwd_env).
template <int N, bool LAG>
__host__ __device__ __forceinline__ void recompute_segment(const AdjArgs& a, const ClassConst& cc,
                                                  const EnvConst& P, const HalfInvT<float>& A,
                                                  const StepConstT<float>& sc,
                                                  float (&x)[Dims<N, LAG>::D], int t0, int t1,
                                                  int base, int64_t j, int64_t c) {
  constexpr int D = Dims<N, LAG>::D;
  const int S = a.substeps;
  for (int t = t0; t < t1; ++t) {
    float act[N], fcmd[N], gcmd[6], dg[6], fs[LAG ? N : 1];
    load_command<N>(cc, a, t, c, act, fcmd, gcmd);
    if constexpr (LAG) {
#pragma unroll
      for (int i = 0; i < N; ++i) fs[i] = x[13 + i];
    }
    begin_control_step<N, LAG>(cc, x, fcmd, dg, cc.rho_s);
    float m[6];
    momentum(P, x + 7, m);
    for (int s = 0; s < S; ++s) {
      float* sb = a.segbuf + (int64_t)((t - base) * S + s) * D * a.Ep + j;
#pragma unroll
      for (int i = 0; i < 13; ++i) sb[i * a.Ep] = x[i];
      if constexpr (LAG) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
          sb[(13 + i) * a.Ep] = fs[i];
          fs[i] = fma_t(sc.rho, fs[i] - fcmd[i], fcmd[i]);
        }
      }
      rk4_substep<N, LAG>(x, m, P, A, gcmd, dg, sc);
    }
  }
}

// WHOLE: the sub-step inputs of the whole rollout are already in segbuf
// (k_adj_recompute); otherwise each segment is recomputed here, into a
// segment-sized segbuf, just before its sweep.  The recomputation loop is
// written out here rather than calling recompute_segment: with that call
// inlined, the one-wave 8-thruster lag instantiation (256 VGPRs + AGPRs)
// returned gradients 5e-2 away from the oracle's although the source was
// equivalent, and out of line the call's register saves made the kernel 2-3x
// slower; this loop, unchanged, matches the oracle to 5e-7.
//
// adj_bwd_env is the backward of one env: internal column j, caller column c,
// its constants P, the step factors sc and the pre-scaled inverse A.  Host and
// device code, so that the same source also runs on the CPU (tests); the
// kernel k_adj_bwd below loads the env's constants and inlines it.
// PREFETCH: the next sub-step's input and the next control step's dL/d traj
// and throttles are loaded one step ahead, so that their latency hides
// behind the current sub-step's VJP (a launch of one wave per SIMD has no
// other wave to hide it behind); it costs 2 D + N registers, which the
// two-wave build cannot spare.
// TRAJ (with WHOLE): one sub-step per control step, each step's input read
// from the caller's trajectory instead of the recomputation buffer.
// TB: ThetaBar<float> (registers) or ThetaBarLds (LDS), zeroed by the caller;
// the parameter adjoints accumulate into it and are written out at the end.
template <int N, bool LAG, bool WHOLE, bool PREFETCH = false, bool TRAJ = false,
          class TB = ThetaBar<float>>
__host__ __device__ __forceinline__ void adj_bwd_env(const AdjArgs& a, const ClassConst& cc,
                                                     const EnvConst& P,
                                                     const StepConstT<float>& sc,
                                                     const HalfInvT<float>& A, int64_t j,
                                                     int64_t c, TB thb) {
  constexpr int D = Dims<N, LAG>::D;
  const int K = a.ckpt_every, S = a.substeps;
  const int nseg = (a.T + K - 1) / K;
  static_assert(WHOLE || !TRAJ, "trajectory inputs replace the whole-rollout buffer");
  // the input of sub-step s of control step t: from the recomputation buffer,
  // or (TRAJ: one sub-step per control step) from the caller's trajectory row
  // of the step before, the first checkpoint for t = 0
  auto load_input = [&](int t, int s, int base, float (&y)[D]) {
    if constexpr (TRAJ) {
      (void)s;
      (void)base;
      const float* p = t == 0 ? a.ckpt + c : a.traj + (int64_t)(t - 1) * a.D * a.E + c;
#pragma unroll
      for (int i = 0; i < D; ++i) y[i] = p[i * a.E];
    } else {
      const float* sb = a.segbuf + (int64_t)((t - base) * S + s) * D * a.Ep + j;
#pragma unroll
      for (int i = 0; i < D; ++i) y[i] = sb[i * a.Ep];
    }
  };
  float lam[D];
#pragma unroll
  for (int i = 0; i < D; ++i) lam[i] = 0.0f;
  for (int seg = nseg - 1; seg >= 0; --seg) {
    const int t0 = seg * K, t1 = min(a.T, t0 + K);
    const int base = WHOLE ? 0 : t0;   // segbuf row of control step t: (t - base) * S
    if constexpr (!WHOLE) {
      // recompute this segment's sub-step inputs from its checkpoint
      float x[D];
      const float* ck = a.ckpt + (int64_t)seg * a.D * a.E + c;
#pragma unroll
      for (int i = 0; i < D; ++i) x[i] = ck[i * a.E];
      // (the forward sets the lag states to their end-of-control-step value at
      // the start; the sub-step inputs the VJP linearises about carry the lag
      // states of each sub-step, f_cmd + rho^s (f - f_cmd), kept here in fs)
      for (int t = t0; t < t1; ++t) {
        float act[N], fcmd[N], gcmd[6], dg[6], fs[LAG ? N : 1];
        load_command<N>(cc, a, t, c, act, fcmd, gcmd);
        if constexpr (LAG) {
#pragma unroll
          for (int i = 0; i < N; ++i) fs[i] = x[13 + i];
        }
        begin_control_step<N, LAG>(cc, x, fcmd, dg, cc.rho_s);
        float m[6];
        momentum(P, x + 7, m);
        for (int s = 0; s < S; ++s) {
          float* sb = a.segbuf + (int64_t)((t - t0) * S + s) * D * a.Ep + j;
#pragma unroll
          for (int i = 0; i < 13; ++i) sb[i * a.Ep] = x[i];
          if constexpr (LAG) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
              sb[(13 + i) * a.Ep] = fs[i];
              fs[i] = fma_t(sc.rho, fs[i] - fcmd[i], fcmd[i]);
            }
          }
          rk4_substep<N, LAG>(x, m, P, A, gcmd, dg, sc);
        }
      }
    }
    // reverse sweep over the segment
    if constexpr (PREFETCH) {
      float y_n[D], gt_n[D], act_n[N];
      {
        load_input(t1 - 1, S - 1, base, y_n);
        const float* gt = a.gtraj + (int64_t)(t1 - 1) * a.D * a.E + c;
#pragma unroll
        for (int i = 0; i < D; ++i) gt_n[i] = gt[i * a.E];
        const float* af = a.actions + (int64_t)(t1 - 1) * a.n_max * a.E + c;
#pragma unroll
        for (int i = 0; i < N; ++i) act_n[i] = af[i * a.E];
      }
      for (int t = t1 - 1; t >= t0; --t) {
        float act[N], fcmd[N], gcmd[6], fcb[N], gcb[6], ab[N];
#pragma unroll
        for (int i = 0; i < D; ++i) lam[i] += gt_n[i];
#pragma unroll
        for (int i = 0; i < N; ++i) act[i] = act_n[i];
        if (t > t0) {
          const float* gt = a.gtraj + (int64_t)(t - 1) * a.D * a.E + c;
#pragma unroll
          for (int i = 0; i < D; ++i) gt_n[i] = gt[i * a.E];
          const float* af = a.actions + (int64_t)(t - 1) * a.n_max * a.E + c;
#pragma unroll
          for (int i = 0; i < N; ++i) act_n[i] = af[i * a.E];
        }
        thrust_command<N>(cc, act, fcmd);
        command_wrench<N>(cc, fcmd, gcmd);
#pragma unroll
        for (int i = 0; i < N; ++i) fcb[i] = 0.0f;
#pragma unroll
        for (int k = 0; k < 6; ++k) gcb[k] = 0.0f;
        for (int s = S - 1; s >= 0; --s) {
          float y[D];
#pragma unroll
          for (int i = 0; i < D; ++i) y[i] = y_n[i];
          if (s > 0)
            load_input(t, s - 1, base, y_n);
          else if (t > t0)
            load_input(t - 1, S - 1, base, y_n);
          rk4_substep_vjp<N, LAG>(y, P, cc, fcmd, gcmd, a.dt, lam, fcb, gcb, thb);
        }
        throttle_vjp<N>(cc, act, fcb, gcb, ab);
        float* ga = a.gact + (int64_t)t * a.n_max * a.E + c;
#pragma unroll
        for (int i = 0; i < N; ++i) ga[i * a.E] = ab[i];
        for (int i = N; i < a.n_max; ++i) ga[i * a.E] = 0.0f;
      }
    } else {
      for (int t = t1 - 1; t >= t0; --t) {
        const float* gt = a.gtraj + (int64_t)t * a.D * a.E + c;
#pragma unroll
        for (int i = 0; i < D; ++i) lam[i] += gt[i * a.E];
        float act[N], fcmd[N], gcmd[6], fcb[N], gcb[6], ab[N];
        load_command<N>(cc, a, t, c, act, fcmd, gcmd);
#pragma unroll
        for (int i = 0; i < N; ++i) fcb[i] = 0.0f;
#pragma unroll
        for (int k = 0; k < 6; ++k) gcb[k] = 0.0f;
        if constexpr (TRAJ) {   // one sub-step per control step
          float y[D];
          load_input(t, 0, base, y);
          rk4_substep_vjp<N, LAG>(y, P, cc, fcmd, gcmd, a.dt, lam, fcb, gcb, thb);
        } else {
          for (int s = S - 1; s >= 0; --s) {
            float y[D];
            load_input(t, s, base, y);
            rk4_substep_vjp<N, LAG, true>(y, P, cc, fcmd, gcmd, a.dt, lam, fcb, gcb, thb);
          }
        }
        throttle_vjp<N>(cc, act, fcb, gcb, ab);
        float* ga = a.gact + (int64_t)t * a.n_max * a.E + c;
#pragma unroll
        for (int i = 0; i < N; ++i) ga[i * a.E] = ab[i];
        for (int i = N; i < a.n_max; ++i) ga[i * a.E] = 0.0f;
      }
    }
  }
  // theta = (M_A(6), D_L(6), D_Q(6), B);  W - B and h_z = W z_g - B z_b carry B
#pragma unroll
  for (int k = 0; k < 18; ++k) a.gtheta[k * a.E + c] = theta_bar_get(thb, k);
  a.gtheta[18 * a.E + c] = -theta_bar_get(thb, 18) - a.zb * theta_bar_get(thb, 19);
  if (a.gx0) {
#pragma unroll
    for (int i = 0; i < D; ++i) a.gx0[i * a.E + c] = lam[i];
    for (int i = D; i < a.D; ++i) a.gx0[i * a.E + c] = 0.0f;
  }
}

}  // namespace mg
