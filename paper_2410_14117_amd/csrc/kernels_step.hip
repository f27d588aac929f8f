// kernels_step.hip -- reset (per-env factorisation), fused / plain step,
// deterministic episode statistics, and layout gather/scatter kernels.
#include "fossen_quad.h"

namespace mg {

// ---------------------------------------------------------------------------
// statistics: wavefront butterfly -> one partial per block (fixed order)
// ---------------------------------------------------------------------------

__device__ __forceinline__ void block_stats(double s_dist, double m_dist, double s_ke,
                                            double n_bad, double* __restrict__ out) {
  __shared__ double sh[kBlock / 64][4];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    s_dist += __shfl_xor(s_dist, off, 64);
    m_dist = fmax(m_dist, __shfl_xor(m_dist, off, 64));
    s_ke += __shfl_xor(s_ke, off, 64);
    n_bad += __shfl_xor(n_bad, off, 64);
  }
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0) {
    sh[wave][0] = s_dist;
    sh[wave][1] = m_dist;
    sh[wave][2] = s_ke;
    sh[wave][3] = n_bad;
  }
  __syncthreads();
  if (threadIdx.x < 4) {
    const int k = threadIdx.x;
    double acc = sh[0][k];
#pragma unroll
    for (int wv = 1; wv < kBlock / 64; ++wv) acc = (k == 1) ? fmax(acc, sh[wv][k]) : acc + sh[wv][k];
    out[k] = acc;
  }
  __syncthreads();
}

// 1/2 nu^T M nu = 1/2 (v . a + w . b), every FMA explicit, so that the kernels
// that form it agree bitwise
__device__ __forceinline__ double kinetic_energy(const EnvConst& P, const float* x) {
  const double u = x[7], v = x[8], w = x[9], p = x[10], q = x[11], r = x[12];
  const double au = fma((double)P.Muu, u, mul_nc((double)P.Muq, q));
  const double av = fma((double)P.Mvv, v, mul_nc((double)P.Mvp, p));
  const double aw = mul_nc((double)P.Mww, w);
  const double bp = fma((double)P.Mvp, v, mul_nc((double)P.Mpp, p));
  const double bq = fma((double)P.Muq, u, mul_nc((double)P.Mqq, q));
  const double br = mul_nc((double)P.Mrr, r);
  return 0.5 * fma(r, br, fma(q, bq, fma(p, bp, fma(w, aw, fma(u, au, mul_nc(v, av))))));
}

// ---------------------------------------------------------------------------
// the step kernel: n_ctrl control steps x substeps RK4 sub-steps per launch,
// state and per-env constants in registers throughout; one env per lane.
// PLAIN instantiations do exactly one sub-step of one control step per launch
// (the per-sub-step comparator whose state round-trips HBM).
// ---------------------------------------------------------------------------

#ifndef MG_STEP_WAVES_PER_EU
#define MG_STEP_WAVES_PER_EU 0
#endif
#if MG_STEP_WAVES_PER_EU > 0
#define MG_STEP_ATTR __attribute__((amdgpu_waves_per_eu(MG_STEP_WAVES_PER_EU)))
#else
#define MG_STEP_ATTR
#endif

template <int N, bool LAG, bool PLAIN>
__global__ void __launch_bounds__(kBlock) MG_STEP_ATTR k_step(const StepArgs a, const ClassConst cc) {
  constexpr int D = Dims<N, LAG>::D;
  const int n_ctrl = PLAIN ? 1 : a.n_ctrl;
  const int substeps = PLAIN ? 1 : a.substeps;
  const int64_t local = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  bool active = local < a.seg_len &&
                MG_CHECK(a, a.seg_start + a.seg_len <= a.Ep, kDbgSegment);
  const int64_t j = a.seg_start + (active ? local : 0);
  // byte offsets of the lane's env in internal and caller rows (rows of at most
  // 2^30 floats, checked by the launcher): every access below is a wave-uniform
  // row pointer plus this 32-bit offset, which the compiler addresses as an
  // SGPR base plus a VGPR offset, with no per-access 64-bit index arithmetic
  const uint32_t jo = (uint32_t)j * 4u;
  int64_t c = active ? (a.perm ? (int64_t)lane_elem(a.perm, jo) : j) : 0;
  active = active && MG_CHECK(a, c >= 0 && c < a.dbg.cols, kDbgColumn);
  c = active ? c : 0;
  const uint32_t co = (uint32_t)c * 4u;

  float x[D];
  EnvConst P;
  // an env whose flags are set is frozen: it is not stepped; an env whose
  // state is non-finite at the end of the launch gets its launch-input state
  // back and is flagged, so that it is frozen from the next launch on
  bool frozen = false;
  if (active) {
#pragma unroll
    for (int i = 0; i < D; ++i) x[i] = lane_elem(a.state + i * a.Ep, jo);
    P = load_env_const_off(a.derived, a.Ep, jo);
    frozen = lane_elem(a.flags, (uint32_t)j) != 0;
  }
  const StepConstT<float> sc = make_step_const(cc, a.dt);
  const HalfInvT<float> A = half_step_inverse(P, sc.h2);
  for (int t = 0; t < n_ctrl; ++t) {
    double s_dist = 0.0, m_dist = 0.0, s_ke = 0.0, n_bad = 0.0;
    if (active) {
      const float* af = a.actions + (int64_t)t * a.n_max * a.E;
      float act[N], fcmd[N], gcmd[6];
#pragma unroll
      for (int i = 0; i < N; ++i) act[i] = lane_elem(af + i * a.E, co);
      thrust_command<N>(cc, act, fcmd);
      command_wrench<N>(cc, fcmd, gcmd);
      if (!frozen)
        control_step<N, LAG>(x, P, A, cc, fcmd, gcmd, sc, substeps, PLAIN ? cc.rho : cc.rho_s);
      if (a.traj) {
        float* tf = a.traj + (int64_t)t * a.D * a.E;
#pragma unroll
        for (int i = 0; i < D; ++i) lane_elem(tf + i * a.E, co) = x[i];
        for (int i = D; i < a.D; ++i) lane_elem(tf + i * a.E, co) = 0.0f;
      }
      if (a.partials) {
        bool finite = !frozen;
#pragma unroll
        for (int i = 0; i < D; ++i) finite = finite && isfinite(x[i]);
        if (finite) {
          float tx = 0.f, ty = 0.f, tz = 0.f;
          if (a.targets) {
            tx = lane_elem(a.targets, co);
            ty = lane_elem(a.targets + a.E, co);
            tz = lane_elem(a.targets + 2 * a.E, co);
          }
          const double dx = (double)x[0] - tx, dy = (double)x[1] - ty, dz = (double)x[2] - tz;
          s_dist = sqrt(fma(dz, dz, fma(dx, dx, mul_nc(dy, dy))));
          m_dist = s_dist;
          s_ke = kinetic_energy(P, x);
        } else {
          n_bad = 1.0;
        }
      }
    }
    if (a.partials)
      block_stats(s_dist, m_dist, s_ke, n_bad,
                  a.partials + ((int64_t)t * a.nblk_total + a.blk_off + blockIdx.x) * 4);
  }
  if (active) {
    bool finite = true;
#pragma unroll
    for (int i = 0; i < D; ++i) finite = finite && isfinite(x[i]);
    if (finite) {
#pragma unroll
      for (int i = 0; i < D; ++i) lane_elem(a.state + i * a.Ep, jo) = x[i];
    } else {
      // the launch-input state stays in place
      lane_elem(a.flags, (uint32_t)j) =
          (uint8_t)(lane_elem(a.flags, (uint32_t)j) | kFlagNonFinite);
    }
  }
}

// The control steps of all classes in one launch: one tail of blocks for all of
// them, no fork and join between class streams, and whole rollouts in one launch
// (a.each).  All classes have a lag or none has; N is the most thrusters of any.
// The class constants and the row pointers are formed anew at each use (the
// pins): held in scalar registers across the control steps they spill, which
// took 20 us of a control step of 2^20 envs.  168 VGPRs, none spilled; of the
// scalar registers 57 (8 lagged thrusters; 40 without a lag) still go to vector
// lanes, none in the sub-step loop: with the largest class's thrusters it makes a
// control step cost about 95 VALU and 185 scalar instructions more than k_step's.
// ORDER: the launch's blocks in the order segs.order gives (ClassSegs), in kernels
// of their own: with the order looked up in every launch seven more scalar registers
// were spilled, and 6 control steps of 16 sub-steps of 2^20 envs of two classes in
// halves took 1139 us against 1097 without it (with the kernels apart, on another
// card, 1054 against 1053).
// Which calls it is used for: one_launch (runtime.hip).  Per control step, before
// (a launch per class and control step, forked and joined or replayed from a graph)
// and with all in one launch, lagged envs, alternating runs: two classes, one call
// per control step with statistics, 131072 envs of 4 sub-steps 48 -> 17.0 us, 2^20
// of 16 187 -> 180; rollouts of 20, 4 sub-steps, 131072 envs 14.0 -> 9.4, 2^20 68
// -> 63; 16 sub-steps, 131072 envs 26.6 -> 24.7, 2^20 168 -> 176 (such calls keep a
// launch per class); one class, 2^20 envs, 4 sub-steps 74 -> 62, 16 sub-steps 176 ->
// 175.  A single class's mg_step stays with k_step, which is 2-8 % faster there.
template <int N, bool LAG, bool ORDER>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3)))
k_step_classes(const StepArgs a, const ClassSegs segs) {
  constexpr int D = Dims<N, LAG>::D;
  int block;
  const int k = block_class(segs, ORDER ? launch_block(segs.order, blockIdx.x) : blockIdx.x, block);
  const ClassConst* ccp = segs.cc + k;
  auto class_const = [&]() { return scalar_class_const(pin_sgpr(ccp)); };
  const int64_t seg_start = segs.start[k], seg_len = segs.len[k];
  const int n = class_const().n_thr;
  const int Dc = LAG ? 13 + n : 13;    // the class's rows
  const int64_t local = (int64_t)block * kBlock + threadIdx.x;
  bool active = local < seg_len && MG_CHECK(a, seg_start + seg_len <= a.Ep, kDbgSegment);
  const int64_t j = seg_start + (active ? local : 0);
  const uint32_t jo = (uint32_t)j * 4u;
  int64_t c = active ? (a.perm ? (int64_t)lane_elem(a.perm, jo) : j) : 0;
  active = active && MG_CHECK(a, c >= 0 && c < a.dbg.cols, kDbgColumn);
  c = active ? c : 0;
  const uint32_t co = (uint32_t)c * 4u;

  float x[D];
  auto load_state = [&]() {
    const float* st = pin_sgpr(a.state);
    const int64_t ld = pin_sgpr(a.Ep);
#pragma unroll
    for (int i = 0; i < D; ++i) x[i] = lane_elem(i < 13 || i < Dc ? st + i * ld : st, jo);
  };
  auto mask_state = [&]() {
#pragma unroll
    for (int i = 13; i < D; ++i) x[i] = i < Dc ? x[i] : 0.0f;
  };
  auto store_state = [&]() {
    float* st = pin_sgpr(a.state);
    const int64_t ld = pin_sgpr(a.Ep);
#pragma unroll
    for (int i = 0; i < 13; ++i) lane_elem(st + i * ld, jo) = x[i];
    if (Dc == D) {
#pragma unroll
      for (int i = 13; i < D; ++i) lane_elem(st + i * ld, jo) = x[i];
    } else {
#pragma unroll
      for (int i = 13; i < D; ++i)
        if (i < Dc) lane_elem(st + i * ld, jo) = x[i];
    }
  };
  auto all_finite = [&]() {
    bool finite = true;
#pragma unroll
    for (int i = 0; i < D; ++i) finite = finite && isfinite(x[i]);
    return finite;
  };
  auto set_nonfinite = [&]() {
    lane_elem(a.flags, (uint32_t)j) =
        (uint8_t)(lane_elem(a.flags, (uint32_t)j) | kFlagNonFinite);
  };
  EnvConst P;
  // an env whose flags are set is frozen: it is not stepped; an env whose
  // state is non-finite at the end of the launch (a.each: of a control step)
  // gets its input state back and is flagged, so that it is frozen from the
  // next launch (control step) on: bad_at is that step
  bool frozen = false;
  int bad_at = a.n_ctrl;
  // each control step's throttles are loaded one step ahead: loads and stores
  // complete in order, so a load behind the trajectory's stores would wait for
  // them
  float nxt[N];
  if (active) {
    load_state();
    P = load_env_const_off(a.derived, pin_sgpr(a.Ep), jo);
    frozen = lane_elem(a.flags, (uint32_t)j) != 0;
    load_throttles<N>(n, a.actions, pin_sgpr(a.E), co, nxt);
    mask_state();
  }
  const StepConstT<float> sc = make_step_const(class_const(), a.dt);
  const HalfInvT<float> A = half_step_inverse(P, sc.h2);
  for (int t = 0; t < a.n_ctrl; ++t) {
    double s_dist = 0.0, m_dist = 0.0, s_ke = 0.0, n_bad = 0.0;
    if (active) {
      const ClassConst cc = class_const();
      float fcmd[N], gcmd[6];
      mask_throttles<N>(n, nxt);
      thrust_command<N>(cc, nxt, fcmd);
      command_wrench<N>(cc, fcmd, gcmd);
      if (t + 1 < a.n_ctrl)
        load_throttles<N>(n, pin_sgpr(a.actions + (int64_t)(t + 1) * a.n_max * a.E),
                          pin_sgpr(a.E), co, nxt);
      if (!frozen)
        control_step<N, LAG>(x, P, A, cc, fcmd, gcmd, sc, a.substeps, cc.rho_s);
      if (a.traj && bad_at == a.n_ctrl) {
        float* tf = pin_sgpr(a.traj + (int64_t)t * a.D * a.E);
        const int64_t ld = pin_sgpr(a.E);
#pragma unroll
        for (int i = 0; i < D; ++i) lane_elem(tf + i * ld, co) = x[i];   // D == a.D
      }
      const bool finite = (a.partials || a.each) ? all_finite() : true;
      if (a.partials) {
        if (finite && !frozen) {
          float tx = 0.f, ty = 0.f, tz = 0.f;
          if (a.targets) {
            tx = lane_elem(a.targets, co);
            ty = lane_elem(a.targets + a.E, co);
            tz = lane_elem(a.targets + 2 * a.E, co);
          }
          const double dx = (double)x[0] - tx, dy = (double)x[1] - ty, dz = (double)x[2] - tz;
          s_dist = sqrt(fma(dz, dz, fma(dx, dx, mul_nc(dy, dy))));
          m_dist = s_dist;
          s_ke = kinetic_energy(P, x);
        } else {
          n_bad = 1.0;
        }
      }
      if (a.each) {
        if (!finite) {
          bad_at = min(bad_at, t);
          frozen = true;
        } else if (!frozen) {
          store_state();
        }
      }
    }
    if (a.partials)
      block_stats(s_dist, m_dist, s_ke, n_bad,
                  a.partials + ((int64_t)t * a.nblk_total +
                                (ORDER ? launch_block(pin_sgpr(segs.order), blockIdx.x)
                                       : blockIdx.x)) * 4);
  }
  if (!active) return;
  if (!a.each && all_finite()) {
    store_state();
  } else if (!a.each || bad_at < a.n_ctrl) {
    set_nonfinite();        // the input state stays in place
    if (!a.traj) return;
    load_state();
    mask_state();
    for (int t = bad_at + 1; t < a.n_ctrl; ++t) {
      float* tf = a.traj + (int64_t)t * a.D * a.E + c;
#pragma unroll
      for (int i = 0; i < D; ++i) tf[i * a.E] = x[i];
    }
  }
}

template <int N, bool LAG>
static hipError_t launch_step_t(const ClassConst& cc, const StepArgs& a, hipStream_t s) {
  const int64_t nblk = (a.seg_len + kBlock - 1) / kBlock;
  if (nblk == 0) return hipSuccess;
  // 32-bit lane offsets (mg_create caps n_envs below 2^30)
  if (a.Ep > ((int64_t)1 << 30) || a.E > ((int64_t)1 << 30)) return hipErrorInvalidValue;
  if (a.n_ctrl == 1 && a.substeps == 1)
    hipLaunchKernelGGL((k_step<N, LAG, true>), dim3((unsigned)nblk), dim3(kBlock), 0, s, a, cc);
  else
    hipLaunchKernelGGL((k_step<N, LAG, false>), dim3((unsigned)nblk), dim3(kBlock), 0, s, a, cc);
  return hipGetLastError();
}

hipError_t launch_step(const ClassConst& cc, const StepArgs& a, hipStream_t s) {
  const bool lag = cc.lag != 0;
#define MG_CASE(n)                                                         \
  case n:                                                                  \
    return lag ? launch_step_t<n, true>(cc, a, s) : launch_step_t<n, false>(cc, a, s);
  switch (cc.n_thr) {
    MG_CASE(1) MG_CASE(2) MG_CASE(3) MG_CASE(4) MG_CASE(5) MG_CASE(6) MG_CASE(7) MG_CASE(8)
    default:
      return hipErrorInvalidValue;
  }
#undef MG_CASE
}

hipError_t launch_step_classes(const ClassSegs& segs, const StepArgs& a, bool lag,
                               hipStream_t s) {
  const int nblk = segs.blk_end[segs.n - 1];
  if (nblk == 0) return hipSuccess;
  if (a.Ep > ((int64_t)1 << 30) || a.E > ((int64_t)1 << 30)) return hipErrorInvalidValue;
  if (a.D != 13 + (lag ? a.n_max : 0)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)nblk), block(kBlock);
#define MG_LAUNCH(N, LAG)                                                               \
  if (segs.order)                                                                       \
    hipLaunchKernelGGL((k_step_classes<N, LAG, true>), grid, block, 0, s, a, segs);     \
  else                                                                                  \
    hipLaunchKernelGGL((k_step_classes<N, LAG, false>), grid, block, 0, s, a, segs);
#define MG_CASE(n)                                                                      \
  case n:                                                                               \
    if (lag) {                                                                          \
      MG_LAUNCH(n, true)                                                                \
    } else {                                                                            \
      MG_LAUNCH(n, false)                                                               \
    }                                                                                   \
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

// ---------------------------------------------------------------------------
// the same control steps with one env per quad of lanes (fossen_quad.h), all
// classes in one launch: launches too small to fill the GPU with one env per
// lane, which last as long as one wave's instruction chain.
// ---------------------------------------------------------------------------

// one control step
template <bool LAG>
__global__ void __launch_bounds__(kQuadBlock) k_step_quad(const StepArgs a, const ClassSegs segs) {
  const int lane = threadIdx.x;
  // the four lanes of a quad share every condition below, so a DPP exchange
  // never reads a lane that is switched off
  const QuadEnv env = quad_env(a, segs, blockIdx.x, lane);
  const ClassConst* __restrict__ cc = segs.cc + env.cls;
  const QuadLane L = quad_lane(lane);
  const int c = L.c, ci = c > 1 ? c - 1 : 0;
  bool active = env.active;
  const uint32_t j = env.j;
  const uint32_t j4 = j * 4u;
  int64_t col = active ? (a.perm ? (int64_t)lane_elem(a.perm, j4) : (int64_t)j) : 0;
  active = active && MG_CHECK(a, col >= 0 && col < a.dbg.cols, kDbgColumn);
  const uint32_t c4 = active ? (uint32_t)col * 4u : 0u;
  const uint32_t s4 = (uint32_t)a.Ep * 4u, e4 = (uint32_t)a.E * 4u;
  const uint32_t ji = j4 + (uint32_t)ci * s4, jc = j4 + (uint32_t)c * s4;   // internal rows
  const uint32_t oi = c4 + (uint32_t)ci * e4, oc = c4 + (uint32_t)c * e4;   // caller rows

  QuadThr th;
  load_quad_thr(cc, c, th);
  const int n_f = th.lag ? th.n : 0;     // lag states of this class
  const QuadPair fs = quad_pair(c, n_f, j4, s4);   // lag states, internal rows
  const QuadPair ta = quad_pair(c, th.n, c4, e4);  // throttles, caller rows
  QuadState x;
  x.p = lane_elem(a.state, ji);
  x.q = lane_elem(a.state + 3 * a.Ep, jc);
  x.v = lane_elem(a.state + 7 * a.Ep, ji);
  x.w = lane_elem(a.state + 10 * a.Ep, ji);
  x.f[0] = x.f[1] = 0.0f;
  if constexpr (LAG) quad_load_pair(fs, a.state + 13 * a.Ep, x.f);
  bool frozen = lane_elem(a.flags, j) != 0;
  const QuadStep sc = quad_step_const(cc, a.dt);
  QuadConst C;
  QuadMass M;
  load_quad_const(a.derived, a.Ep, j4, c, sc.h2, C, M);
  float act[2];
  quad_load_pair(ta, a.actions, act);
  float tg = 0.0f;
  if (a.partials && a.targets) tg = lane_elem(a.targets, oi);
  if constexpr (LAG) quad_mask_pair(fs, x.f);
  quad_mask_pair(ta, act);
  if (!frozen) quad_control_step<LAG>(L, C, M, th, sc, act, x, a.substeps);
  if (a.traj && active) {
    lane_elem(a.traj + 3 * a.E, oc) = x.q;
    if (c > 0) {
      lane_elem(a.traj, oi) = x.p;
      lane_elem(a.traj + 7 * a.E, oi) = x.v;
      lane_elem(a.traj + 10 * a.E, oi) = x.w;
    }
    if constexpr (LAG) {   // zeros past the class's own
      if (13 + c < a.D) lane_elem(a.traj + 13 * a.E, oc) = x.f[0];
      if (17 + c < a.D) lane_elem(a.traj + 17 * a.E, oc) = x.f[1];
    }
  }
  int finite = isfinite(x.q) && isfinite(x.f[0]) && isfinite(x.f[1]) &&
               (c == 0 || (isfinite(x.p) && isfinite(x.v) && isfinite(x.w)));
  finite &= qperm<MG_QP(1, 0, 3, 2)>(finite);
  finite &= qperm<MG_QP(2, 3, 0, 1)>(finite);
  if (a.partials) {
    const double s = quad_stats(c, M, x.p, x.v, x.w, tg, active, active && finite && !frozen);
    if (lane < 4) a.partials[(int64_t)blockIdx.x * 4 + lane] = s;
  }
  if (!active) return;
  if (finite) {
    lane_elem(a.state + 3 * a.Ep, jc) = x.q;
    if (c > 0) {
      lane_elem(a.state, ji) = x.p;
      lane_elem(a.state + 7 * a.Ep, ji) = x.v;
      lane_elem(a.state + 10 * a.Ep, ji) = x.w;
    }
    if constexpr (LAG) quad_store_pair(fs, a.state + 13 * a.Ep, x.f);
  } else if (c == 0) {   // the input state stays in place
    lane_elem(a.flags, j) = (uint8_t)(lane_elem(a.flags, j) | kFlagNonFinite);
  }
}

// Several control steps in two waves per 16 envs.  Only the rigid-body state is
// serial through the sub-steps; the commands and lag states of the control steps
// ahead, and the rows and statistics of those behind, are not.  Wave 0 takes the
// sub-steps; in phase t, while it takes control step t, wave 1 writes what step
// t - 1 left and forms the wrenches of step t + 1, through LDS; n_ctrl + 1 phases
// for both waves alike.  The values are those of k_step_quad, bitwise.  4096
// Heavies, 200 control steps of 4 sub-steps with trajectory and statistics: 551 us
// in one wave, 403 here, where the sub-steps are 0.50 us each; the adjoint's
// forward of 16 control steps, 8192 envs, 17.5 -> 14.0 us (one sub-step, no lag)
// and 42 -> 37 us (four, lag).
// MODE: frozen as one launch, frozen as one launch per control step, or the
// adjoint's forward (nothing frozen; checkpoints).
enum { kRollLaunch, kRollEach, kRollAdjoint };

template <bool LAG, int MODE>
__global__ void __launch_bounds__(2 * kQuadBlock) k_roll_quad(const StepArgs a,
                                                              const ClassSegs segs, float* ckpt,
                                                              int ckpt_every) {
  __shared__ float4 cmd[2][kQuadBlock];   // command wrench and lag wrench of a control step
  __shared__ float4 out[2][kQuadBlock];   // position, quaternion, velocities after it
  __shared__ int status[2][kQuadBlock];   // 1: frozen before it, 2: non-finite after it
  __shared__ int lag_ok[2][kQuadBlock];   // the lane's thruster states are finite after it
  constexpr bool kLagOk = LAG && MODE != kRollAdjoint;
  const int lane = threadIdx.x & (kQuadBlock - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kQuadBlock);
  // the four lanes of a quad share every condition below
  const QuadEnv env = quad_env(a, segs, blockIdx.x, lane);
  const ClassConst* __restrict__ cc = segs.cc + env.cls;
  const QuadLane L = quad_lane(lane);
  const int c = L.c, ci = c > 1 ? c - 1 : 0;
  bool active = env.active;
  const uint32_t j = env.j, j4 = j * 4u;
  const int64_t col = active ? (a.perm ? (int64_t)lane_elem(a.perm, j4) : (int64_t)j) : 0;
  active = active && MG_CHECK(a, col >= 0 && col < a.dbg.cols, kDbgColumn);
  const uint32_t c4 = active ? (uint32_t)col * 4u : 0u;
  const uint32_t s4 = (uint32_t)a.Ep * 4u, e4 = (uint32_t)a.E * 4u;
  const uint32_t ji = j4 + (uint32_t)ci * s4, jc = j4 + (uint32_t)c * s4;   // internal rows
  const uint32_t oi = c4 + (uint32_t)ci * e4, oc = c4 + (uint32_t)c * e4;   // caller rows
  const QuadStep sc = quad_step_const(cc, a.dt);
  QuadConst C;
  QuadMass M;
  load_quad_const(a.derived, a.Ep, j4, c, sc.h2, C, M);
  bool frozen = MODE != kRollAdjoint && lane_elem(a.flags, j) != 0;
  QuadState x;
  x.p = lane_elem(a.state, ji);
  x.q = lane_elem(a.state + 3 * a.Ep, jc);
  x.v = lane_elem(a.state + 7 * a.Ep, ji);
  x.w = lane_elem(a.state + 10 * a.Ep, ji);
  x.f[0] = x.f[1] = 0.0f;
  const int n = a.n_ctrl;
  if (wave == 0) {
    bool bad = false;
    for (int t = 0; t < n; ++t) {
      lds_barrier();
      const float4 u = cmd[t & 1][lane];
      int f_ok = 1;
      if constexpr (kLagOk) f_ok = lag_ok[t & 1][lane];
      const QuadState x0 = x;
      const int was = frozen ? 1 : 0;
      if (!frozen) {
        float dl = u.z, da = u.w, ml, ma;
        quad_momentum(M, x.v, x.w, ml, ma);
        for (int i = 0; i < a.substeps; ++i)
          quad_substep<LAG>(L, C, sc, x, ml, ma, u.x, u.y, dl, da);
      }
      out[t & 1][lane] = make_float4(x.p, x.q, x.v, x.w);
      if constexpr (MODE != kRollAdjoint) {
        int ok = 1;
        if (MODE == kRollEach || t == n - 1) {
          ok = f_ok && isfinite(x.q) &&
               (c == 0 || (isfinite(x.p) && isfinite(x.v) && isfinite(x.w)));
          ok &= qperm<MG_QP(1, 0, 3, 2)>(ok);
          ok &= qperm<MG_QP(2, 3, 0, 1)>(ok);
        }
        status[t & 1][lane] = was | (ok ? 0 : 2);
        if (!ok) {
          bad = true;
          if constexpr (MODE == kRollEach) {
            x = x0;
            frozen = true;
          }
        }
      }
    }
    lds_barrier();
    if (!active) return;
    if (bad && c == 0)
      lane_elem(a.flags, j) = (uint8_t)(lane_elem(a.flags, j) | kFlagNonFinite);
    if (bad && MODE == kRollLaunch) return;   // the launch-input state stays in place
    lane_elem(a.state + 3 * a.Ep, jc) = x.q;
    if (c > 0) {
      lane_elem(a.state, ji) = x.p;
      lane_elem(a.state + 7 * a.Ep, ji) = x.v;
      lane_elem(a.state + 10 * a.Ep, ji) = x.w;
    }
    return;
  }
  QuadThr th;
  load_quad_thr(cc, c, th);
  const QuadPair fs = quad_pair(c, th.lag ? th.n : 0, j4, s4);   // lag states, internal rows
  const QuadPair ta = quad_pair(c, th.n, c4, e4);                // throttles, caller rows
  if constexpr (LAG) quad_load_pair(fs, a.state + 13 * a.Ep, x.f);
  const int64_t frame = (int64_t)a.n_max * a.E;
  float nxt[2];   // throttles, loaded one control step ahead of their use
  quad_load_pair(ta, a.actions, nxt);
  float tg = 0.0f;
  if (a.partials && a.targets) tg = lane_elem(a.targets, oi);
  if constexpr (LAG) quad_mask_pair(fs, x.f);
  // lag states before the control step that wave 0 has finished, after it, after
  // the next, and of an env that is frozen
  float f0[2] = {0.0f, 0.0f}, f1[2] = {0.0f, 0.0f}, ff[2] = {x.f[0], x.f[1]};
  int last = frozen ? 1 : 0;
  auto prepare = [&](int t) {
    float act[2] = {nxt[0], nxt[1]};
    quad_mask_pair(ta, act);
    if (t + 1 < n) quad_load_pair(ta, a.actions + (int64_t)(t + 1) * frame, nxt);
    f0[0] = f1[0];
    f0[1] = f1[1];
    f1[0] = x.f[0];
    f1[1] = x.f[1];
    float gl, ga, dl, da;
    quad_command<LAG>(th, act, th.rho_s, x, gl, ga, dl, da);
    cmd[t & 1][lane] = make_float4(gl, ga, dl, da);
    // (an env frozen part-way has its flag already; one frozen from the start
    // keeps its thruster states)
    if constexpr (kLagOk)
      lag_ok[t & 1][lane] = frozen ? isfinite(ff[0]) && isfinite(ff[1])
                                   : isfinite(x.f[0]) && isfinite(x.f[1]);
  };
  auto store = [&](float* rows, const float4& u, const float (&f)[2]) {
    if (!active) return;
    lane_elem(rows + 3 * a.E, oc) = u.y;
    if (c > 0) {
      lane_elem(rows, oi) = u.x;
      lane_elem(rows + 7 * a.E, oi) = u.z;
      lane_elem(rows + 10 * a.E, oi) = u.w;
    }
    if constexpr (LAG) {   // zeros past the class's own
      if (13 + c < a.D) lane_elem(rows + 13 * a.E, oc) = f[0];
      if (17 + c < a.D) lane_elem(rows + 17 * a.E, oc) = f[1];
    }
  };
  int until = ckpt_every;   // control steps to the next checkpoint
  // fi, fo: lag states before and after control step t
  auto finish = [&](int t, const float (&fi)[2], const float (&fo)[2]) {
    const float4 u = out[t & 1][lane];
    const int st = MODE != kRollAdjoint ? status[t & 1][lane] : 0;
    last = st;
    const bool was = (st & 1) != 0;
    const float f[2] = {was ? ff[0] : fo[0], was ? ff[1] : fo[1]};
    if (a.traj) store(a.traj + (int64_t)t * a.D * a.E, u, f);
    if constexpr (MODE == kRollAdjoint) {
      if (--until == 0) {
        ckpt += a.D * a.E;
        until = ckpt_every;
        if (t + 1 < n) store(ckpt, u, f);
      }
    }
    if (a.partials) {
      int ok = isfinite(u.y) && isfinite(f[0]) && isfinite(f[1]) &&
               (c == 0 || (isfinite(u.x) && isfinite(u.z) && isfinite(u.w)));
      ok &= qperm<MG_QP(1, 0, 3, 2)>(ok);
      ok &= qperm<MG_QP(2, 3, 0, 1)>(ok);
      const double s = quad_stats(c, M, u.x, u.z, u.w, tg, active, active && ok && !was);
      if (lane < 4) a.partials[((int64_t)t * a.nblk_total + blockIdx.x) * 4 + lane] = s;
    }
    if constexpr (MODE == kRollEach) {
      if (!was && (st & 2)) {   // frozen from here on at the step's input
        ff[0] = fi[0];
        ff[1] = fi[1];
      }
    }
  };
  if constexpr (MODE == kRollAdjoint) store(ckpt, make_float4(x.p, x.q, x.v, x.w), x.f);
  prepare(0);
  for (int t = 0; t < n; ++t) {
    lds_barrier();
    if (t > 0) finish(t - 1, f0, f1);
    if (t + 1 < n) prepare(t + 1);
  }
  lds_barrier();
  finish(n - 1, f1, x.f);
  if constexpr (LAG) {
    if (!active || (MODE == kRollLaunch && (last & 2))) return;
    const float f[2] = {last ? ff[0] : x.f[0], last ? ff[1] : x.f[1]};
    quad_store_pair(fs, a.state + 13 * a.Ep, f);
  }
}

template <int MODE>
static void launch_roll(const ClassSegs& q, const StepArgs& a, bool lag, float* ckpt,
                        int32_t ckpt_every, hipStream_t s) {
  const dim3 grid((unsigned)q.blk_end[q.n - 1]), block(2 * kQuadBlock);
  if (lag)
    hipLaunchKernelGGL((k_roll_quad<true, MODE>), grid, block, 0, s, a, q, ckpt, ckpt_every);
  else
    hipLaunchKernelGGL((k_roll_quad<false, MODE>), grid, block, 0, s, a, q, ckpt, ckpt_every);
}

hipError_t launch_step_quad(const ClassSegs& q, const StepArgs& a, bool lag, bool each_step,
                            hipStream_t s) {
  const int nblk = q.blk_end[q.n - 1];
  if (nblk == 0) return hipSuccess;
  if (a.Ep > kQuadMaxEnvs || a.E > kQuadMaxEnvs) return hipErrorInvalidValue;
  const dim3 grid((unsigned)nblk), block(kQuadBlock);
  // (frozen at the launch's input and at the control step's are the same for one)
  if (a.n_ctrl > 1 && each_step)
    launch_roll<kRollEach>(q, a, lag, nullptr, 1, s);
  else if (a.n_ctrl > 1)
    launch_roll<kRollLaunch>(q, a, lag, nullptr, 1, s);
  else if (lag)
    hipLaunchKernelGGL((k_step_quad<true>), grid, block, 0, s, a, q);
  else
    hipLaunchKernelGGL((k_step_quad<false>), grid, block, 0, s, a, q);
  return hipGetLastError();
}

hipError_t launch_forward_quad(const ClassSegs& q, const StepArgs& a, bool lag, float* ckpt,
                               int32_t ckpt_every, hipStream_t s) {
  if (a.Ep > kQuadMaxEnvs || a.E > kQuadMaxEnvs) return hipErrorInvalidValue;
  launch_roll<kRollAdjoint>(q, a, lag, ckpt, ckpt_every, s);
  return hipGetLastError();
}

// second pass: stats[t] = fixed-order combination of the per-block partials
__global__ void __launch_bounds__(256) k_stats_finalize(const double* __restrict__ partials,
                                                        int32_t nblk, double* __restrict__ stats) {
  const int t = blockIdx.x;
  const double* p = partials + (int64_t)t * nblk * 4;
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  for (int b = threadIdx.x; b < nblk; b += 256) {
    v[0] += p[b * 4 + 0];
    v[1] = fmax(v[1], p[b * 4 + 1]);
    v[2] += p[b * 4 + 2];
    v[3] += p[b * 4 + 3];
  }
  __shared__ double sh[256][4];
#pragma unroll
  for (int k = 0; k < 4; ++k) sh[threadIdx.x][k] = v[k];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      sh[threadIdx.x][0] += sh[threadIdx.x + w][0];
      sh[threadIdx.x][1] = fmax(sh[threadIdx.x][1], sh[threadIdx.x + w][1]);
      sh[threadIdx.x][2] += sh[threadIdx.x + w][2];
      sh[threadIdx.x][3] += sh[threadIdx.x + w][3];
    }
    __syncthreads();
  }
  if (threadIdx.x < 4) stats[t * 4 + threadIdx.x] = sh[0][threadIdx.x];
}

hipError_t launch_stats_finalize(const double* partials, int32_t nblk, int32_t n_ctrl,
                                 double* stats, hipStream_t s) {
  if (n_ctrl <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_stats_finalize, dim3(n_ctrl), dim3(256), 0, s, partials, nblk, stats);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// reset: parameters (nominal x multiplier, or absolute), the per-env
// factorisation of M = M_RB + M_A (FP64, rounded once), and the state
// ---------------------------------------------------------------------------

// Bandwidth-bound: 23 + D floats in, 53 + D out per env; 2^20 Heavies 132 -> 105 us
// (4.7 TB/s, a large copy's rate) since every load precedes the first store.  A
// reset of every env of interleaved classes goes through them in internal order
// (a.perm), so that it is the reads that are scattered and not the writes, or in
// caller order: reset_internal (runtime.hip).
__global__ void __launch_bounds__(256) k_reset(const ResetArgs a) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t k = t, j;       // column of the inputs, internal index
  if (!a.ids && a.perm) {
    if (t >= a.Ep) return;
    k = a.perm[t];
    j = t;
    if (k < 0) return;    // padding
    if (!MG_CHECK(a, k < a.dbg.cols, kDbgColumn)) return;
  } else {
    if (t >= a.n) return;
    const int64_t id = a.ids ? a.ids[k] : k;
    if (id < 0 || id >= a.E) return;   // out-of-range ids are skipped (documented)
    if (!MG_CHECK(a, id < a.dbg.cols, kDbgColumn)) return;
    j = a.iperm ? (int64_t)a.iperm[id] : id;
    if (!MG_CHECK(a, j >= 0 && j < a.Ep, kDbgInternal)) return;
  }
  const ClassNominal& nom = a.nominal[a.class_of[j]];
  // the state is loaded before set_env_params, whose stores no load may pass
  constexpr int kMaxD = 13 + kMaxThr;
  float x[kMaxD];
  if (a.write_state) {
    const int Dc = 13 + (nom.lag ? nom.n_thr : 0);
#pragma unroll
    for (int i = 0; i < kMaxD; ++i) {
      x[i] = i == 3 ? 1.0f : 0.0f;
      if (a.state_in && i < a.D) x[i] = a.state_in[i * a.n + k];
    }
#pragma unroll
    for (int i = 13; i < kMaxD; ++i) x[i] = i < Dc ? x[i] : 0.0f;
  }
  const bool spd = set_env_params(nom, a.param_in ? a.param_in + k : nullptr, a.n,
                                  a.param_absolute != 0, a.params, a.derived, a.Ep, j);
  if (a.flags) {
    const uint8_t keep = a.write_state ? 0 : (uint8_t)(a.flags[j] & kFlagNonFinite);
    a.flags[j] = (uint8_t)(keep | (spd ? 0 : kFlagNotSPD));
  }
  if (!a.write_state) return;
  if (a.task_k) a.task_k[j] = 0;
  if (a.split_acc)
    for (int i = 0; i < 6; ++i) a.split_acc[i * a.Ep + j] = 0.0f;
#pragma unroll
  for (int i = 0; i < kMaxD; ++i)
    if (i < a.D) a.state[i * a.Ep + j] = x[i];
}

hipError_t launch_reset(const ResetArgs& a, hipStream_t s) {
  if (a.n <= 0) return hipSuccess;
  const int64_t nblk = ((!a.ids && a.perm ? a.Ep : a.n) + 255) / 256;
  hipLaunchKernelGGL(k_reset, dim3((unsigned)nblk), dim3(256), 0, s, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// internal <-> caller order (blockIdx.y: kGatherRows rows at a time, so that their
// loads are in flight together)
// ---------------------------------------------------------------------------

constexpr int kGatherRows = 8;

// One caller env per thread (iperm: caller -> internal): interleaved classes are
// read as a few consecutive streams and written as one.
__global__ void __launch_bounds__(256) k_gather_out(const float* __restrict__ in, int64_t Ep,
                                                    float* __restrict__ out, int64_t E,
                                                    int32_t rows,
                                                    const int32_t* __restrict__ iperm) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= E) return;
  const int64_t j = iperm ? (int64_t)iperm[c] : c;
  const int r0 = blockIdx.y * kGatherRows;
#pragma unroll
  for (int r = r0; r < r0 + kGatherRows; ++r)
    if (r < rows) out[r * E + c] = in[r * Ep + j];
}

template <int ROWS>
__global__ void __launch_bounds__(256) k_scatter_in(const float* __restrict__ in, int64_t E,
                                                    float* __restrict__ out, int64_t Ep,
                                                    int32_t rows,
                                                    const int32_t* __restrict__ perm,
                                                    int64_t n_internal) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n_internal) return;
  const int64_t c = perm ? (int64_t)perm[j] : j;
  if (c < 0 || c >= E) return;
  const int r0 = blockIdx.y * ROWS;
#pragma unroll
  for (int r = r0; r < r0 + ROWS; ++r)
    if (r < rows) out[r * Ep + j] = in[r * E + c];
}

// status flags, internal bytes -> caller int32
__global__ void k_flags_out(const uint8_t* __restrict__ flags, int32_t* __restrict__ out,
                            int64_t E, const int32_t* __restrict__ perm, int64_t n_internal) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n_internal) return;
  const int64_t c = perm ? (int64_t)perm[j] : j;
  if (c < 0 || c >= E) return;
  out[c] = flags[j];
}

// flags &= mask for every env
__global__ void k_flags_mask(uint8_t* __restrict__ flags, int64_t n, uint8_t mask) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j < n) flags[j] = (uint8_t)(flags[j] & mask);
}

hipError_t launch_flags_out(const uint8_t* flags, int32_t* out, int64_t E, const int32_t* perm,
                            int64_t n_internal, hipStream_t s) {
  if (n_internal <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_flags_out, dim3((unsigned)((n_internal + 255) / 256)), dim3(256), 0, s,
                     flags, out, E, perm, n_internal);
  return hipGetLastError();
}

hipError_t launch_flags_mask(uint8_t* flags, int64_t n, uint8_t mask, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_flags_mask, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, flags, n,
                     mask);
  return hipGetLastError();
}

static dim3 gather_grid(int64_t n, int32_t rows, int32_t at_a_time = kGatherRows) {
  return dim3((unsigned)((n + 255) / 256), (unsigned)((rows + at_a_time - 1) / at_a_time));
}

hipError_t launch_gather_out(const float* in, int64_t Ep, float* out, int64_t E, int32_t rows,
                             const int32_t* iperm, hipStream_t s) {
  hipLaunchKernelGGL(k_gather_out, gather_grid(E, rows), dim3(256), 0, s, in, Ep, out, E, rows,
                     iperm);
  return hipGetLastError();
}

hipError_t launch_scatter_in(const float* in, int64_t E, float* out, int64_t Ep, int32_t rows,
                             const int32_t* perm, int64_t n_internal, int32_t n_classes,
                             hipStream_t s) {
  if (n_internal <= 0) return hipSuccess;
  // more than two classes read parts of the same lines at different times; where
  // kGatherRows rows are more than an L2 keeps meanwhile and one is not, all rows in
  // one thread (8 classes: 300 000 envs 24.3 -> 21.8 us, 140 000 and 500 000 level;
  // 16 classes: 40.4 -> 31.7; 2 classes, 140 000 to 300 000: 8.0-14.0 against 10.9-15.0)
  constexpr int kAllRows = 24;
  if (n_classes > 2 && rows <= kAllRows && E > 196608 && E <= 524288)
    hipLaunchKernelGGL((k_scatter_in<kAllRows>), gather_grid(n_internal, rows, kAllRows), dim3(256),
                       0, s, in, E, out, Ep, rows, perm, n_internal);
  else
    hipLaunchKernelGGL((k_scatter_in<kGatherRows>), gather_grid(n_internal, rows), dim3(256), 0, s,
                       in, E, out, Ep, rows, perm, n_internal);
  return hipGetLastError();
}

}  // namespace mg
