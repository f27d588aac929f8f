// kernels_task.hip -- Gym-style task step of Sec. III: one control step of
// the fused sub-step loop followed by the task epilogue (the error of Eq. (4),
// episode end, automatic reset, the observation of Eq. (2)), or the
// observation alone, for all classes in one launch.  One env per lane, or per
// quad of lanes (fossen_quad.h) for launches of at most one wave per SIMD; the
// epilogue works in FP64 from the FP32 state and writes FP32.
#include "fossen_quad.h"

namespace mg {

namespace {

constexpr double kPi = 3.1415926535897932384626433832795;

// Reference point p_r and the horizontal direction (vx, vy) of the reference
// heading, given sin and cos of the curve parameter s = omega t + phase.  For
// the circle and the helix the reference velocity is omega R (-sin s, cos s);
// for the lemniscate of Bernoulli R (cos s, sin s cos s) / (1 + sin^2 s) it is
// omega R (-sin s (3 - sin^2 s), 1 - 3 sin^2 s) / (1 + sin^2 s)^2 (the positive
// factor R / (1 + sin^2 s)^2 drops out of the direction).  Station keeping:
// the centre, headed along the target yaw.
__device__ __forceinline__ void reference(const TaskConst& tc, const double (&c)[3], double yaw,
                                          double t, double sn, double cs, double (&pr)[3],
                                          double& vx, double& vy) {
  if (tc.task == 0) {
    pr[0] = c[0];
    pr[1] = c[1];
    pr[2] = c[2];
    float sy, cy;
    sincosf((float)yaw, &sy, &cy);
    vx = cy;
    vy = sy;
    return;
  }
  if (tc.task == 3) {
    const double s2 = mul_nc(sn, sn), inv = 1.0 / (1.0 + s2);
    pr[0] = c[0] + tc.R * cs * inv;
    pr[1] = c[1] + tc.R * sn * cs * inv;
    pr[2] = c[2];
    vx = -tc.omega * sn * (3.0 - s2);
    vy = tc.omega * (1.0 - 3.0 * s2);
  } else {
    pr[0] = c[0] + tc.R * cs;
    pr[1] = c[1] + tc.R * sn;
    pr[2] = c[2] + (tc.task == 2 ? tc.climb * t : 0.0);
    vx = -tc.omega * sn;
    vy = tc.omega * cs;
  }
}

// ZYX roll and pitch of the attitude (w, x, y, z) from the third row of R(q):
// roll = atan2(R32, R33), pitch = atan2(-R31, |(R32, R33)|) (well conditioned at
// any pitch, unlike asin(-R31) near +-90 deg), and the body's horizontal heading
// (hx, hy) = R(q) e1, parallel to (cos yaw, sin yaw) while |pitch| < 90 deg.
struct Attitude {
  float roll, pitch;
  double hx, hy;
};
__device__ __forceinline__ Attitude attitude(float w, float qx, float qy, float qz) {
  Attitude t;
  const float r32 = 2.0f * (w * qx + qy * qz), r33 = 1.0f - 2.0f * (qx * qx + qy * qy);
  const float r31 = 2.0f * (qx * qz - w * qy);
  t.roll = atan2f(r32, r33);
  if (t.roll <= -3.14159265f) t.roll = 3.14159265f;
  t.pitch = atan2f(-r31, sqrtf(r32 * r32 + r33 * r33));
  t.hx = 1.0 - 2.0 * ((double)qy * qy + (double)qz * qz);
  t.hy = 2.0 * ((double)qx * qy + (double)w * qz);
  return t;
}

// The curve parameters of the look-ahead points follow one another by the
// rotation (cos, sin)(omega dl).
__device__ __forceinline__ void next_point(const TaskConst& tc, double& sn, double& cs) {
  const double sn1 = fma(sn, tc.cdl, mul_nc(cs, tc.sdl));
  cs = fma(cs, tc.cdl, mul_nc(-sn, tc.sdl));
  sn = sn1;
}

// The six rows of look-ahead point i (time t since the episode's start, curve
// parameter's sin and cos at the point) at o, row stride E.  The heading error
// wrap(yaw - yaw_r) is the signed angle from the reference direction to the
// body's heading, one atan2.
__device__ __forceinline__ void observe_point(const TaskConst& tc, const float (&p)[3],
                                              const Attitude& at, const double (&c)[3], double yaw,
                                              double t, int i, double sn, double cs, float* o,
                                              int64_t E) {
  double pr[3], vx, vy;
  reference(tc, c, yaw, fma((double)(i + 1), tc.dl, t), sn, cs, pr, vx, vy);
  float herr = atan2f((float)(at.hy * vx - at.hx * vy), (float)(at.hx * vx + at.hy * vy));
  if (herr <= -3.14159265f) herr = 3.14159265f;
  o[0] = (float)(p[0] - pr[0]);
  o[E] = (float)(p[1] - pr[1]);
  o[2 * E] = (float)(p[2] - pr[2]);
  o[3 * E] = at.roll;
  o[4 * E] = at.pitch;
  o[5 * E] = herr;
}

// Position error of Eq. (4).
__device__ __forceinline__ double position_error(const float (&p)[3], const double (&pr)[3]) {
  const double dx = p[0] - pr[0], dy = p[1] - pr[1], dz = p[2] - pr[2];
  return sqrt(fma(dz, dz, fma(dx, dx, mul_nc(dy, dy))));
}

// sin and cos of the curve parameter s = omega t + phase: s is formed and
// reduced to [-pi, pi] in FP64, then evaluated in FP32 (errors ~1e-7, well
// inside the observation's FP32 output).
__device__ __forceinline__ void curve_sincos(const TaskConst& tc, double t, double phase,
                                             double& sn, double& cs) {
  if (tc.task == 0) {
    sn = 0.0;
    cs = 1.0;
    return;
  }
  const double s = fma(tc.omega, t, phase);
  const double r = s - (2.0 * kPi) * rint(s * (0.5 / kPi));
  float sf, cf;
  sincosf((float)r, &sf, &cf);
  sn = sf;
  cs = cf;
}

}  // namespace

// Held to three resident waves per SIMD (at most 168 VGPRs), the step kernel's
// occupancy: left to itself the compiler gives the 8-thruster lag variant more
// registers for the epilogue, which leaves room for two waves only.  N is the
// most thrusters of any class and LAG whether any class has a lag.  One launch
// for all classes instead of one each, forked and joined through events: 7 task
// steps of 57 059 interleaved envs with reset and read-back 436 -> 167 us, 9 of
// 214 719 703 -> 555 us, 2 of 2^20 with 16 sub-steps 620 -> 610 us.
// A sim of one class takes its constants from the kernel's arguments (OneClass): read
// through memory, and with the selects for smaller classes, a task step of 20 000 to
// 300 000 envs took 4-16 % longer, an observation 3-18 %.
template <int N, bool LAG, class SEGS>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3)))
k_task(const TaskArgs a, const SEGS segs, const TaskConst tc) {
  constexpr int D = Dims<N, LAG>::D;
  const BlockClass<SEGS> cls(segs, blockIdx.x);
  const int64_t local = (int64_t)cls.block * kBlock + threadIdx.x;
  if (local >= cls.len) return;
  if (!MG_CHECK(a, cls.start + cls.len <= a.Ep, kDbgSegment)) return;
  const int64_t j = cls.start + local;
  const uint32_t jo = (uint32_t)j * 4u;
  const int64_t c = a.perm ? (int64_t)lane_elem(a.perm, jo) : j;
  if (!MG_CHECK(a, c >= 0 && c < a.dbg.cols, kDbgColumn)) return;
  const uint32_t co = (uint32_t)c * 4u;
  float x[D];
  int n = N, Dc = D;   // the class's thrusters and rows
  if constexpr (!cls.kOne) {
    const ClassConst cc = cls.first_constants();
    n = cc.n_thr;
    Dc = 13 + (LAG && cc.lag ? n : 0);
  }
#pragma unroll
  for (int i = 0; i < D; ++i)
    x[i] = lane_elem(i < 13 || i < Dc ? a.state + i * a.Ep : a.state, jo);
  int32_t k = lane_elem(a.task_k, jo);
  if (a.actions) {
    const EnvConst P = load_env_const_off(a.derived, a.Ep, jo);
    const ClassConst cc = cls.constants();
    float act[N], fcmd[N], gcmd[6];
    load_throttles<N>(n, a.actions, a.E, co, act);
    const StepConstT<float> sc = make_step_const(cc, a.dt);
    const HalfInvT<float> A = half_step_inverse(P, sc.h2);
    mask_throttles<N>(n, act);
    thrust_command<N>(cc, act, fcmd);
    command_wrench<N>(cc, fcmd, gcmd);
    // rows past the class's: at their commands, so that they have no lag wrench
    // (their columns of B are zero, or the class has no lag)
#pragma unroll
    for (int i = 13; i < D; ++i) x[i] = i < Dc ? x[i] : fcmd[i - 13];
    control_step<N, LAG>(x, P, A, cc, fcmd, gcmd, sc, a.substeps,
                         a.substeps == 1 ? cc.rho : cc.rho_s);
    k += 1;
  }
#pragma unroll
  for (int i = 13; i < D; ++i) x[i] = i < Dc ? x[i] : 0.0f;
  // the task's per-env data is read after the sub-steps, so that it does not
  // occupy registers across them
  const float* tf = pin_sgpr(a.task_f);
  const int64_t ld = pin_sgpr(a.Ep);
  const double cen[3] = {lane_elem(tf, jo), lane_elem(tf + ld, jo), lane_elem(tf + 2 * ld, jo)};
  const double phase = lane_elem(tf + 3 * ld, jo), yaw = lane_elem(tf + 4 * ld, jo);
  // sin and cos of the curve parameter at the current episode time
  double sn, cs;
  curve_sincos(tc, k * tc.dtc, phase, sn, cs);
  if (a.actions) {
    bool finite = true;
#pragma unroll
    for (int i = 0; i < D; ++i) finite = finite && isfinite(x[i]);
    double pr[3], vx, vy;
    reference(tc, cen, yaw, k * tc.dtc, sn, cs, pr, vx, vy);
    const float p[3] = {x[0], x[1], x[2]};
    const double e = position_error(p, pr);
    const bool term = !finite || (tc.emax > 0.0 && !(e <= tc.emax));
    const int32_t d = term ? 1 : (k >= tc.L ? 2 : 0);
    if (a.err) lane_elem(a.err, co) = (float)e;
    if (a.done) lane_elem(a.done, co) = d;
    if (d) {
#pragma unroll
      for (int i = 0; i < D; ++i)
        if (i < 13 || i < Dc)
          x[i] = a.reset_state ? a.reset_state[i * a.E + c] : (i == 3 ? 1.0f : 0.0f);
      k = 0;
      curve_sincos(tc, 0.0, phase, sn, cs);
      uint8_t fl = (uint8_t)(a.flags[j] & kFlagNotSPD);
      if (a.reset_mult)
        fl = set_env_params(a.nominal[cls.k], a.reset_mult + c, a.E, false, a.params, a.derived,
                            a.Ep, j) ? 0 : kFlagNotSPD;
      a.flags[j] = fl;
    }
#pragma unroll
    for (int i = 0; i < D; ++i)
      if (i < 13 || i < Dc) lane_elem(a.state + i * a.Ep, jo) = x[i];
    lane_elem(a.task_k, jo) = k;
  }
  const Attitude at = attitude(x[3], x[4], x[5], x[6]);
  const float p[3] = {x[0], x[1], x[2]};
  const double t = k * tc.dtc;
  const int m = tc.task == 0 ? 1 : tc.m;
  float* o = a.obs + c;
  for (int i = 0; i < m; ++i) {
    next_point(tc, sn, cs);
    observe_point(tc, p, at, cen, yaw, t, i, sn, cs, o + (int64_t)(6 * i) * a.E, a.E);
  }
  o += (int64_t)(6 * m) * a.E;
#pragma unroll
  for (int i = 0; i < 6; ++i) o[i * a.E] = x[7 + i];
}

// The same with one env per quad of lanes: the control step of fossen_quad.h,
// then each lane takes the look-ahead points c, c + 4, ...  (10 task steps of 267
// envs with 16 sub-steps, reset and read-back: 225 -> 189 us.)
template <bool LAG>
__global__ void __launch_bounds__(kQuadBlock) k_task_quad(const TaskArgs a, const ClassSegs segs,
                                                          const TaskConst tc) {
  // the four lanes of a quad share every condition below, but for lane 0's
  // restart of the parameters
  const QuadEnv env = quad_env(a, segs, blockIdx.x, threadIdx.x);
  const int cls = env.cls;
  const ClassConst* __restrict__ cc = segs.cc + cls;
  const QuadLane L = quad_lane(threadIdx.x);
  const int c = L.c, ci = c > 1 ? c - 1 : 0;
  bool active = env.active;
  const uint32_t j = env.j, j4 = j * 4u;
  const int64_t col = active ? (a.perm ? (int64_t)lane_elem(a.perm, j4) : (int64_t)j) : 0;
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
  int32_t k = lane_elem(a.task_k, j4);
  const double cen[3] = {lane_elem(a.task_f, j4), lane_elem(a.task_f + a.Ep, j4),
                         lane_elem(a.task_f + 2 * a.Ep, j4)};
  const double phase = lane_elem(a.task_f + 3 * a.Ep, j4);
  const double yaw = lane_elem(a.task_f + 4 * a.Ep, j4);
  if (a.actions) {
    float act[2];
    quad_load_pair(thr_in, a.actions, act);
    const QuadStep sc = quad_step_const(cc, a.dt);
    QuadConst C;
    QuadMass M;
    load_quad_const(a.derived, a.Ep, j4, c, sc.h2, C, M);
    quad_mask_pair(thr_in, act);
    if constexpr (LAG) quad_mask_pair(fs, x.f);
    quad_control_step<LAG>(L, C, M, th, sc, act, x, a.substeps);
    k += 1;
  }
  double sn, cs;
  curve_sincos(tc, k * tc.dtc, phase, sn, cs);
  auto position = [&](float (&p)[3]) {
    p[0] = qperm<MG_QP(1, 1, 1, 1)>(x.p);
    p[1] = qperm<MG_QP(2, 2, 2, 2)>(x.p);
    p[2] = qperm<MG_QP(3, 3, 3, 3)>(x.p);
  };
  float p[3];
  if (a.actions) {
    int finite = isfinite(x.q) && isfinite(x.f[0]) && isfinite(x.f[1]) &&
                 (c == 0 || (isfinite(x.p) && isfinite(x.v) && isfinite(x.w)));
    finite &= qperm<MG_QP(1, 0, 3, 2)>(finite);
    finite &= qperm<MG_QP(2, 3, 0, 1)>(finite);
    double pr[3], vx, vy;
    reference(tc, cen, yaw, k * tc.dtc, sn, cs, pr, vx, vy);
    position(p);
    const double e = position_error(p, pr);
    const bool term = !finite || (tc.emax > 0.0 && !(e <= tc.emax));
    const int32_t d = term ? 1 : (k >= tc.L ? 2 : 0);
    if (active && c == 0 && a.err) lane_elem(a.err, c4) = (float)e;
    if (active && c == 0 && a.done) lane_elem(a.done, c4) = d;
    if (active && d) {
      x.p = x.v = x.w = x.f[0] = x.f[1] = 0.0f;
      x.q = c == 0 ? 1.0f : 0.0f;
      if (a.reset_state) {
        x.p = lane_elem(a.reset_state, oi);
        x.q = lane_elem(a.reset_state + 3 * a.E, oc);
        x.v = lane_elem(a.reset_state + 7 * a.E, oi);
        x.w = lane_elem(a.reset_state + 10 * a.E, oi);
        if constexpr (LAG) {
          quad_load_pair(quad_pair(c, n_f, c4, e4), a.reset_state + 13 * a.E, x.f);
          quad_mask_pair(fs, x.f);
        }
      }
      k = 0;
      curve_sincos(tc, 0.0, phase, sn, cs);
      if (c == 0) {
        uint8_t fl = (uint8_t)(a.flags[j] & kFlagNotSPD);
        if (a.reset_mult)
          fl = set_env_params(a.nominal[cls], a.reset_mult + c4 / 4u, a.E, false, a.params,
                              a.derived, a.Ep, j) ? 0 : kFlagNotSPD;
        a.flags[j] = fl;
      }
    }
    if (active) {
      lane_elem(a.state + 3 * a.Ep, jc) = x.q;
      if (c > 0) {
        lane_elem(a.state, ji) = x.p;
        lane_elem(a.state + 7 * a.Ep, ji) = x.v;
        lane_elem(a.state + 10 * a.Ep, ji) = x.w;
      } else {
        lane_elem(a.task_k, j4) = k;
      }
      if constexpr (LAG) quad_store_pair(fs, a.state + 13 * a.Ep, x.f);
    }
  }
  position(p);
  const Attitude at = attitude(qperm<MG_QP(0, 0, 0, 0)>(x.q), qperm<MG_QP(1, 1, 1, 1)>(x.q),
                               qperm<MG_QP(2, 2, 2, 2)>(x.q), qperm<MG_QP(3, 3, 3, 3)>(x.q));
  const double t = k * tc.dtc;
  const int m = tc.task == 0 ? 1 : tc.m;
  float* o = a.obs + c4 / 4u;
  for (int i0 = 0; i0 < m; i0 += 4) {
    double sni = sn, csi = cs;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      next_point(tc, sn, cs);
      sni = i == c ? sn : sni;
      csi = i == c ? cs : csi;
    }
    if (active && i0 + c < m)
      observe_point(tc, p, at, cen, yaw, t, i0 + c, sni, csi,
                    o + (int64_t)(6 * (i0 + c)) * a.E, a.E);
  }
  if (active && c > 0) {
    o += (int64_t)(6 * m) * a.E;
    o[ci * a.E] = x.v;
    o[(3 + ci) * a.E] = x.w;
  }
}

hipError_t launch_task(const ClassSegs& segs, const ClassConst& cc, const TaskConst& tc,
                       const TaskArgs& a, bool lag, bool quad, hipStream_t s) {
  const int nblk = segs.blk_end[segs.n - 1];
  if (nblk == 0) return hipSuccess;
  // 32-bit lane offsets: one row, or (quad) every row at once
  const int64_t most = quad ? kQuadMaxEnvs : (int64_t)1 << 30;
  if (a.Ep > most || a.E > most) return hipErrorInvalidValue;
  const dim3 grid((unsigned)nblk), block(kBlock);
  if (quad) {
    if (lag)
      hipLaunchKernelGGL((k_task_quad<true>), grid, dim3(kQuadBlock), 0, s, a, segs, tc);
    else
      hipLaunchKernelGGL((k_task_quad<false>), grid, dim3(kQuadBlock), 0, s, a, segs, tc);
    return hipGetLastError();
  }
  const OneClass one{cc, segs.start[0], segs.len[0]};
#define MG_LAUNCH(N, lagged)                                                                  \
  do {                                                                                        \
    if (segs.n == 1)                                                                          \
      hipLaunchKernelGGL((k_task<N, lagged, OneClass>), grid, block, 0, s, a, one, tc);       \
    else                                                                                      \
      hipLaunchKernelGGL((k_task<N, lagged, ClassSegs>), grid, block, 0, s, a, segs, tc);     \
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
