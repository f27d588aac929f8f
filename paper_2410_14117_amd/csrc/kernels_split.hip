// kernels_split.hip -- the split integration of Sec. II as a variant of the
// step: a physics engine advances the rigid body (M_RB, C_RB, g_RB) while the
// hydrodynamic wrench, computed from the current state, acts on it as an
// external force.  Per sub-step of dt:
//   tau_h = -M_A a_prev - C_A(nu) nu - D(nu) nu - g_A(eta)
//   a     = M_RB^-1 (tau_thrust + tau_h - C_RB(nu) nu - g_RB(eta))
//   nu <- nu + dt a;  p <- p + dt R(q) v;  q <- (q + dt/2 q (x) (0, w)) / |.|
//   f  <- f + dt (f_cmd - f) / tau_thr;  a_prev <- a
// Since C and g are linear in M and in (W, B), tau_h - C_RB nu - g_RB is the
// coupled residual tau - C(M) nu - D nu - g of the fused step minus
// M_A a_prev, so the residual code is shared.
//
// The lag step maps f - f_cmd to kappa (f - f_cmd), kappa = 1 - dt / tau_thr,
// with the command held over a control step, so its wrench B (f - f_cmd) is
// formed once per control step and carried, and the lag states are set to
// their end-of-control-step value f_cmd + kappa^S (f - f_cmd) at its start (kappa^S
// scaled where it is beyond FP32, so that a thruster at rest stays there):
// nothing in a sub-step depends on the thrusters, so one launch serves all
// classes (N is the most thrusters of any; the others' throttles past their own
// are zeros, as are their columns of B).
//
// One env per lane, or per quad of lanes (fossen_quad.h) for launches of at
// most one wave per SIMD, which last as long as one env's chain.
#include "fossen_quad.h"

namespace mg {

namespace {

// M_RB^-1 for r_g on the z axis: (u, q) and (v, p) couple through m z_g.
struct RigidInv {
  float uu, vv, ww, pp, qq, rr, uq, vp;
};

__device__ __forceinline__ RigidInv rigid_inverse(const float* params, int64_t Ep, uint32_t jo,
                                                  double zg) {
  const double m = lane_elem(params, jo), ix = lane_elem(params + Ep, jo),
               iy = lane_elem(params + 2 * Ep, jo), iz = lane_elem(params + 3 * Ep, jo);
  const double mzz = mul_nc(mul_nc(m, zg), zg);
  const double mpp = ix + mzz, mqq = iy + mzz, muq = m * zg, mvp = -m * zg;
  const double det_uq = m * mqq - muq * muq, det_vp = m * mpp - mvp * mvp;
  RigidInv I;
  I.uu = (float)(mqq / det_uq);
  I.qq = (float)(m / det_uq);
  I.uq = (float)(-muq / det_uq);
  I.vv = (float)(mpp / det_vp);
  I.pp = (float)(m / det_vp);
  I.vp = (float)(-mvp / det_vp);
  I.ww = (float)(1.0 / m);
  I.rr = (float)(1.0 / iz);
  return I;
}

}  // namespace

// VALU-bound: 131 instructions per sub-step (211 with 8 thrusters before the lag
// wrench was carried); 105 VGPRs, four waves per SIMD.  The class constants are
// scalars, read anew at each control step: through a plain pointer they were
// vector loads, waited for at each control step, and cost 54 more registers.
// Lagged Heavies, 10 control steps of 16 sub-steps with trajectory, with a launch
// per class and the lag states stepped, and now: 32 768 envs 74 -> 57 us, 131 072
// 109 -> 81, 524 288 400 -> 294.
// A sim of one class takes its constants from the kernel's arguments (OneClass); read
// through memory, short calls of few sub-steps took up to 25 % longer.
template <int N, bool LAG, class SEGS>
__global__ void __launch_bounds__(kBlock) k_split(const SplitArgs a, const SEGS segs) {
  constexpr int D = Dims<N, LAG>::D;
  const BlockClass<SEGS> cls(segs, blockIdx.x);
  int n = N, Dc = D;                     // this class's thrusters and rows
  bool lag = LAG;
  if constexpr (!cls.kOne) {
    n = cls.first_constants().n_thr;
    lag = LAG && cls.first_constants().lag;
    Dc = 13 + (lag ? n : 0);
  }
  const int64_t local = (int64_t)cls.block * kBlock + threadIdx.x;
  if (local >= cls.len) return;
  if (!MG_CHECK(a, cls.start + cls.len <= a.Ep, kDbgSegment)) return;
  const int64_t j = cls.start + local;
  const uint32_t jo = (uint32_t)j * 4u;
  const int64_t c = a.perm ? (int64_t)lane_elem(a.perm, jo) : j;
  if (!MG_CHECK(a, c >= 0 && c < a.dbg.cols, kDbgColumn)) return;
  const uint32_t co = (uint32_t)c * 4u;
  float x[D], acc[6], ma[6];
#pragma unroll
  for (int i = 0; i < D; ++i)
    x[i] = lane_elem(i < 13 || i < Dc ? a.state + i * a.Ep : a.state, jo);
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    acc[i] = lane_elem(a.acc + i * a.Ep, jo);
    ma[i] = lane_elem(a.params + (4 + i) * a.Ep, jo);
  }
  const EnvConst P = load_env_const_off(a.derived, a.Ep, jo);
  // each control step's throttles are loaded one step ahead: loads and stores
  // complete in order, so a load behind the trajectory's stores would wait for
  // them at every control step
  const int64_t frame = (int64_t)a.n_max * a.E;
  float nxt[N];
  load_throttles<N>(n, a.actions, a.E, co, nxt);
  const RigidInv I = rigid_inverse(a.params, a.Ep, jo, a.nominal[cls.k].zg);
  const float dt = to_vgpr(a.dt), hdt = to_vgpr(0.5f * a.dt);
  const float kappa = to_vgpr(cls.first_constants().kappa);
#pragma unroll
  for (int i = 13; i < D; ++i) x[i] = i < Dc ? x[i] : 0.0f;
  for (int t = 0; t < a.n_ctrl; ++t) {
    const ClassConst cc = cls.constants();
    float fcmd[N], gcmd[6], dg[6];
    mask_throttles<N>(n, nxt);
    thrust_command<N>(cc, nxt, fcmd);
    command_wrench<N>(cc, fcmd, gcmd);
    if (t + 1 < a.n_ctrl)
      load_throttles<N>(n, pin_sgpr(a.actions + (int64_t)(t + 1) * frame), pin_sgpr(a.E), co, nxt);
#pragma unroll
    for (int i = 0; i < 6; ++i) dg[i] = 0.0f;
    if constexpr (LAG) {
      if (lag) {
        lag_wrench<N>(cc, x, fcmd, dg);
#pragma unroll
        for (int i = 0; i < N; ++i)
          x[13 + i] = fma_t(cc.kappa_s, ldexpf(x[13 + i] - fcmd[i], cc.kappa_e), fcmd[i]);
      }
    }
    for (int s = 0; s < a.substeps; ++s) {
      float tau[6], kin[7], r[6], mom[6];
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        tau[i] = LAG ? gcmd[i] + dg[i] : gcmd[i];
        if constexpr (LAG) dg[i] = mul_nc(dg[i], kappa);
      }
      momentum(P, x + 7, mom);
      rhs_residual_m(x, mom, kin, r, P, tau);
#pragma unroll
      for (int i = 0; i < 6; ++i) r[i] = fma_t(-ma[i], acc[i], r[i]);
      acc[0] = fma_t(I.uq, r[4], I.uu * r[0]);
      acc[1] = fma_t(I.vp, r[3], I.vv * r[1]);
      acc[2] = mul_nc(I.ww, r[2]);
      acc[3] = fma_t(I.pp, r[3], I.vp * r[1]);
      acc[4] = fma_t(I.qq, r[4], I.uq * r[0]);
      acc[5] = mul_nc(I.rr, r[5]);
#pragma unroll
      for (int i = 0; i < 6; ++i) x[7 + i] = fma_t(dt, acc[i], x[7 + i]);
      // kinematics at the new velocities: p += dt R(q) v, q += dt/2 q (x) (0, w)
      rhs_residual_m(x, mom, kin, r, P, tau);
#pragma unroll
      for (int i = 0; i < 3; ++i) x[i] = fma_t(dt, kin[i], x[i]);
#pragma unroll
      for (int i = 3; i < 7; ++i) x[i] = fma_t(hdt, kin[i], x[i]);
      const float inv = rsqrt_t(
          fma_t(x[6], x[6], fma_t(x[5], x[5], fma_t(x[3], x[3], x[4] * x[4]))));
#pragma unroll
      for (int i = 3; i < 7; ++i) x[i] *= inv;
    }
    if (a.traj) {
      float* tf = pin_sgpr(a.traj + (int64_t)t * a.D * a.E);
      const int64_t ld = pin_sgpr(a.E);
#pragma unroll
      for (int i = 0; i < 13; ++i) lane_elem(tf + i * ld, co) = x[i];
      if (D == a.D) {
#pragma unroll
        for (int i = 13; i < D; ++i) lane_elem(tf + i * ld, co) = x[i];
      } else {   // the classes with most thrusters have no lag
#pragma unroll
        for (int i = 13; i < D; ++i)
          if (i < a.D) lane_elem(tf + i * ld, co) = x[i];
      }
    }
  }
#pragma unroll
  for (int i = 0; i < D; ++i)
    if (i < 13 || i < Dc) lane_elem(a.state + i * a.Ep, jo) = x[i];
#pragma unroll
  for (int i = 0; i < 6; ++i) lane_elem(a.acc + i * a.Ep, jo) = acc[i];
}

#pragma clang fp contract(off)

// The same with one env per quad of lanes, bitwise: launches of at most one
// wave per SIMD (16 384 envs: 71 -> 38 us, 1000 envs: 69 -> 32 us as above; at
// two waves per SIMD it would be level with one env per lane).
template <bool LAG>
__global__ void __launch_bounds__(kQuadBlock) k_split_quad(const SplitArgs a,
                                                           const ClassSegs segs) {
  // the four lanes of a quad share every condition below
  const QuadEnv env = quad_env(a, segs, blockIdx.x, threadIdx.x);
  const int k = env.cls;
  const ClassConst* __restrict__ cc = segs.cc + k;
  const QuadLane L = quad_lane(threadIdx.x);
  const int c = L.c, ci = c > 1 ? c - 1 : 0;
  bool active = env.active;
  const uint32_t j4 = env.j * 4u;
  const int64_t col = active ? (a.perm ? (int64_t)lane_elem(a.perm, j4) : (int64_t)env.j) : 0;
  active = active && MG_CHECK(a, col >= 0 && col < a.dbg.cols, kDbgColumn);
  const uint32_t c4 = active ? (uint32_t)col * 4u : 0u;
  const uint32_t s4 = (uint32_t)a.Ep * 4u, e4 = (uint32_t)a.E * 4u;
  const uint32_t ji = j4 + (uint32_t)ci * s4, jc = j4 + (uint32_t)c * s4;   // internal rows
  const uint32_t oi = c4 + (uint32_t)ci * e4, oc = c4 + (uint32_t)c * e4;   // caller rows
  QuadThr th;
  load_quad_thr(cc, c, th);
  const int n_f = th.lag ? th.n : 0;
  const QuadPair fs = quad_pair(c, n_f, j4, s4);     // lag states, internal rows
  const QuadPair thr_in = quad_pair(c, th.n, c4, e4);  // throttles, caller rows
  QuadState x;
  x.p = lane_elem(a.state, ji);
  x.q = lane_elem(a.state + 3 * a.Ep, jc);
  x.v = lane_elem(a.state + 7 * a.Ep, ji);
  x.w = lane_elem(a.state + 10 * a.Ep, ji);
  x.f[0] = x.f[1] = 0.0f;
  if constexpr (LAG) quad_load_pair(fs, a.state + 13 * a.Ep, x.f);
  float al = lane_elem(a.acc, ji), aa = lane_elem(a.acc + 3 * a.Ep, ji);
  const float mal = lane_elem(a.params + 4 * a.Ep, ji), maa = lane_elem(a.params + 7 * a.Ep, ji);
  QuadConst C;
  QuadMass M;
  load_quad_const(a.derived, a.Ep, j4, c, 1.0f, C, M);
  const RigidInv I = rigid_inverse(a.params, a.Ep, j4, a.nominal[k].zg);
  const float il = c == 1 ? I.uu : (c == 2 ? I.vv : I.ww);
  const float ia = c == 1 ? I.pp : (c == 2 ? I.qq : I.rr);
  const float icl = c == 1 ? I.uq : (c == 2 ? I.vp : 0.0f);
  const float ica = c == 1 ? I.vp : (c == 2 ? I.uq : 0.0f);
  const float dt = to_vgpr(a.dt), hdt = to_vgpr(0.5f * a.dt), kappa = to_vgpr(cc->kappa);
  const int64_t frame = (int64_t)a.n_max * a.E;
  float nxt[2];   // throttles, loaded one control step ahead
  quad_load_pair(thr_in, a.actions, nxt);
  if constexpr (LAG) quad_mask_pair(fs, x.f);
  for (int t = 0; t < a.n_ctrl; ++t) {
    float act[2] = {nxt[0], nxt[1]};
    quad_mask_pair(thr_in, act);
    if (t + 1 < a.n_ctrl) quad_load_pair(thr_in, a.actions + (int64_t)(t + 1) * frame, nxt);
    float gl, ga, dl, da;
    quad_command<LAG, true>(th, act, cc->kappa_s, x, gl, ga, dl, da, cc->kappa_e);
    for (int s = 0; s < a.substeps; ++s) {
      const float tl = LAG ? gl + dl : gl, ta = LAG ? ga + da : ga;
      if constexpr (LAG) {
        dl *= kappa;
        da *= kappa;
      }
      float ml, ma, rl, ra, kp, kq;
      quad_momentum(M, x.v, x.w, ml, ma);
      quad_forces(L, C, x.q, x.v, x.w, ml, ma, tl, ta, rl, ra);
      rl = fmaf(-mal, al, rl);
      ra = fmaf(-maa, aa, ra);
      al = fmaf(qperm<kSwapXY>(ra), icl, il * rl);
      aa = fmaf(ia, ra, qperm<kSwapXY>(rl) * ica);
      x.v = fmaf(dt, al, x.v);
      x.w = fmaf(dt, aa, x.w);
      quad_kinematics(L, x.q, x.v, x.w, kp, kq);
      x.p = fmaf(dt, kp, x.p);
      x.q = quad_normalise(fmaf(hdt, kq, x.q));
    }
    if (a.traj && active) {
      float* tf = a.traj + (int64_t)t * a.D * a.E;
      lane_elem(tf + 3 * a.E, oc) = x.q;
      if (c > 0) {
        lane_elem(tf, oi) = x.p;
        lane_elem(tf + 7 * a.E, oi) = x.v;
        lane_elem(tf + 10 * a.E, oi) = x.w;
      }
      if constexpr (LAG) {   // zeros past the class's own
        if (13 + c < a.D) lane_elem(tf + 13 * a.E, oc) = x.f[0];
        if (17 + c < a.D) lane_elem(tf + 17 * a.E, oc) = x.f[1];
      }
    }
  }
  if (!active) return;
  lane_elem(a.state + 3 * a.Ep, jc) = x.q;
  if (c > 0) {
    lane_elem(a.state, ji) = x.p;
    lane_elem(a.state + 7 * a.Ep, ji) = x.v;
    lane_elem(a.state + 10 * a.Ep, ji) = x.w;
    lane_elem(a.acc, ji) = al;
    lane_elem(a.acc + 3 * a.Ep, ji) = aa;
  }
  if constexpr (LAG) quad_store_pair(fs, a.state + 13 * a.Ep, x.f);
}

#pragma clang fp contract(fast)

hipError_t launch_split(const ClassSegs& segs, const ClassConst& cc, const SplitArgs& a, bool lag,
                        bool quad, hipStream_t s) {
  const int nblk = segs.blk_end[segs.n - 1];
  if (nblk == 0) return hipSuccess;
  // 32-bit lane offsets: one row, or (quad) every row at once
  const int64_t most = quad ? kQuadMaxEnvs : (int64_t)1 << 30;
  if (a.Ep > most || a.E > most) return hipErrorInvalidValue;
  const dim3 grid((unsigned)nblk);
  if (quad && lag)
    hipLaunchKernelGGL((k_split_quad<true>), grid, dim3(kQuadBlock), 0, s, a, segs);
  else if (quad)
    hipLaunchKernelGGL((k_split_quad<false>), grid, dim3(kQuadBlock), 0, s, a, segs);
  if (quad) return hipGetLastError();
  const dim3 block(kBlock);
  const OneClass one{cc, segs.start[0], segs.len[0]};
#define MG_LAUNCH(N, lagged)                                                                  \
  do {                                                                                        \
    if (segs.n == 1)                                                                          \
      hipLaunchKernelGGL((k_split<N, lagged, OneClass>), grid, block, 0, s, a, one);          \
    else                                                                                      \
      hipLaunchKernelGGL((k_split<N, lagged, ClassSegs>), grid, block, 0, s, a, segs);        \
  } while (0)
#define MG_CASE(n)       \
  case n:                \
    if (lag)             \
      MG_LAUNCH(n, true); \
    else                 \
      MG_LAUNCH(n, false); \
    break;
  switch (a.n_max) {
    MG_CASE(1) MG_CASE(2) MG_CASE(3) MG_CASE(4) MG_CASE(5) MG_CASE(6) MG_CASE(7) MG_CASE(8)
    default:
      return hipErrorInvalidValue;
  }
#undef MG_CASE
#undef MG_LAUNCH
  return hipGetLastError();
}

}  // namespace mg
