// kernels_adjoint_quad.hip -- the adjoint's kernels with one env per quad of
// lanes and all classes in one launch (fossen_quad_adjoint.h), for sims too
// small to fill the GPU with one env per lane: a launch then lasts as long as
// one env's chain of sub-steps (at 2.1 ns an instruction for a lone wave), which
// is 1.4 times shorter here forward and 1.6-1.7 times backward.  Results are
// bitwise those of kernels_adjoint.hip.  Forward and backward with all that goes
// with them, one env per lane and now: 8192 envs without lag, 64 control steps of
// one sub-step 336 -> 210 us; 3001 envs with lag, 32 control steps of four
// sub-steps 639 -> 365 us.
#include "fossen_quad_adjoint.h"

namespace mg {

namespace {

// A lane's place: its class, env and component, and the byte offsets of its
// rows (row pointers are wave-uniform; every row of a state within 4 GiB).
struct QuadPlace {
  int cls, c;
  bool active;          // all four lanes of a quad alike
  uint32_t j4, c4;      // internal and caller column
  uint32_t ji, jc, oi, oc;   // 3-vector and quaternion rows, internal and caller
};

__device__ __forceinline__ QuadPlace quad_place(const ClassSegs& segs, const AdjArgs& a) {
  QuadPlace p;
  int k = 0;
  while (k + 1 < segs.n && (int)blockIdx.x >= segs.blk_end[k]) ++k;
  const int blk0 = k > 0 ? segs.blk_end[k - 1] : 0;
  p.cls = k;
  p.c = threadIdx.x & 3;
  const int ci = p.c > 1 ? p.c - 1 : 0;
  const int64_t local = (int64_t)((int)blockIdx.x - blk0) * kQuadEnvs + (threadIdx.x >> 2);
  p.active = local < segs.len[k] &&
             MG_CHECK(a, segs.start[k] + segs.len[k] <= a.Ep, kDbgSegment);
  p.j4 = (uint32_t)(segs.start[k] + (p.active ? local : 0)) * 4u;
  const int64_t col =
      p.active ? (a.perm ? (int64_t)lane_elem(a.perm, p.j4) : (int64_t)(p.j4 / 4u)) : 0;
  p.active = p.active && MG_CHECK(a, col >= 0 && col < a.dbg.cols, kDbgColumn);
  p.c4 = p.active ? (uint32_t)col * 4u : 0u;
  const uint32_t s4 = (uint32_t)a.Ep * 4u, e4 = (uint32_t)a.E * 4u;
  p.ji = p.j4 + (uint32_t)ci * s4;
  p.jc = p.j4 + (uint32_t)p.c * s4;
  p.oi = p.c4 + (uint32_t)ci * e4;
  p.oc = p.c4 + (uint32_t)p.c * e4;
  return p;
}

// One state's rows, row stride ld floats; lane offsets vi (3-vectors), vc.
__device__ __forceinline__ void quad_load_state(const float* rows, int64_t ld, uint32_t vi,
                                                uint32_t vc, bool f0, bool f1, QuadState& x) {
  x.q = lane_elem(rows + 3 * ld, vc);
  x.v = lane_elem(rows + 7 * ld, vi);
  x.w = lane_elem(rows + 10 * ld, vi);
  x.f[0] = f0 ? lane_elem(rows + 13 * ld, vc) : 0.0f;
  x.f[1] = f1 ? lane_elem(rows + 17 * ld, vc) : 0.0f;
}

// A caller state [D][E]: rows past the class's are zero.
__device__ __forceinline__ void quad_store_caller(float* rows, const AdjArgs& a,
                                                  const QuadPlace& p, bool f0, bool f1, float xp,
                                                  float xq, float xv, float xw, float x0,
                                                  float x1) {
  lane_elem(rows + 3 * a.E, p.oc) = xq;
  if (p.c > 0) {
    lane_elem(rows, p.oi) = xp;
    lane_elem(rows + 7 * a.E, p.oi) = xv;
    lane_elem(rows + 10 * a.E, p.oi) = xw;
  }
  if (13 + p.c < a.D) lane_elem(rows + 13 * a.E, p.oc) = f0 ? x0 : 0.0f;
  if (17 + p.c < a.D) lane_elem(rows + 17 * a.E, p.oc) = f1 ? x1 : 0.0f;
}

__device__ __forceinline__ void quad_load_throttles(const AdjArgs& a, const QuadPlace& p, int n,
                                                    int t, float (&act)[2]) {
  const float* af = a.actions + (int64_t)t * a.n_max * a.E;
  act[0] = p.c < n ? lane_elem(af, p.oc) : 0.0f;
  act[1] = p.c + 4 < n ? lane_elem(af + 4 * a.E, p.oc) : 0.0f;
}

}  // namespace

template <bool LAG>
__global__ void __launch_bounds__(kQuadBlock) k_adj_quad_fwd(const AdjArgs a,
                                                             const ClassSegs segs) {
  const QuadPlace p = quad_place(segs, a);
  const ClassConst* __restrict__ cc = segs.cc + p.cls;
  const QuadLane L = quad_lane(threadIdx.x);
  QuadThr th;
  load_quad_thr(cc, p.c, th);
  const int n_f = th.lag ? th.n : 0;
  const bool f0 = p.c < n_f, f1 = p.c + 4 < n_f;
  QuadState x;
  x.p = lane_elem(a.state, p.ji);
  quad_load_state(a.state, a.Ep, p.ji, p.jc, f0, f1, x);
  const QuadStep sc = quad_step_const(cc, a.dt);
  QuadConst C;
  QuadMass M;
  load_quad_const(a.derived, a.Ep, p.j4, p.c, sc.h2, C, M);
  float nxt[2];
  quad_load_throttles(a, p, th.n, 0, nxt);
  for (int t = 0; t < a.T; ++t) {
    const float act[2] = {nxt[0], nxt[1]};
    if (t + 1 < a.T) quad_load_throttles(a, p, th.n, t + 1, nxt);
    if (p.active && t % a.ckpt_every == 0)
      quad_store_caller(a.ckpt + (int64_t)(t / a.ckpt_every) * a.D * a.E, a, p, f0, f1, x.p, x.q,
                        x.v, x.w, x.f[0], x.f[1]);
    quad_control_step<LAG>(L, C, M, th, sc, act, x, a.substeps);
    if (p.active && a.traj)
      quad_store_caller(a.traj + (int64_t)t * a.D * a.E, a, p, f0, f1, x.p, x.q, x.v, x.w, x.f[0],
                        x.f[1]);
  }
  if (!p.active) return;
  lane_elem(a.state + 3 * a.Ep, p.jc) = x.q;
  if (p.c > 0) {
    lane_elem(a.state, p.ji) = x.p;
    lane_elem(a.state + 7 * a.Ep, p.ji) = x.v;
    lane_elem(a.state + 10 * a.Ep, p.ji) = x.w;
  }
  if (f0) lane_elem(a.state + 13 * a.Ep, p.jc) = x.f[0];
  if (f1) lane_elem(a.state + 17 * a.Ep, p.jc) = x.f[1];
}

// Every segment's sub-step inputs at once (blockIdx.y = segment) into the
// whole-rollout segbuf.  Position rows are left out: the sweep reads none.
template <bool LAG>
__global__ void __launch_bounds__(kQuadBlock) k_adj_quad_recompute(const AdjArgs a,
                                                                   const ClassSegs segs) {
  const QuadPlace p = quad_place(segs, a);
  const ClassConst* __restrict__ cc = segs.cc + p.cls;
  const QuadLane L = quad_lane(threadIdx.x);
  QuadThr th;
  load_quad_thr(cc, p.c, th);
  const int n_f = th.lag ? th.n : 0;
  const bool f0 = p.c < n_f, f1 = p.c + 4 < n_f;
  const int seg = blockIdx.y;
  const int t0 = seg * a.ckpt_every, t1 = min(a.T, t0 + a.ckpt_every);
  const float* src = a.ckpt + (int64_t)seg * a.D * a.E;
  QuadState x;
  x.p = 0.0f;
  quad_load_state(src, a.E, p.oi, p.oc, f0, f1, x);
  const QuadStep sc = quad_step_const(cc, a.dt);
  QuadConst C;
  QuadMass M;
  load_quad_const(a.derived, a.Ep, p.j4, p.c, sc.h2, C, M);
  for (int t = t0; t < t1; ++t) {
    float act[2], fcmd[2], gl, ga, dl, da, ml, ma;
    quad_load_throttles(a, p, th.n, t, act);
    quad_thrust(th, act, fcmd);
    // each sub-step's own lag states, f_cmd + rho^s (f - f_cmd)
    float fs[2] = {x.f[0], x.f[1]};
    quad_begin<LAG>(th, M, act, x, gl, ga, dl, da, ml, ma);
    for (int s = 0; s < a.substeps; ++s) {
      float* sb = a.segbuf + ((int64_t)t * a.substeps + s) * a.D * a.Ep;
      if (p.active) {
        lane_elem(sb + 3 * a.Ep, p.jc) = x.q;
        if (p.c > 0) {
          lane_elem(sb + 7 * a.Ep, p.ji) = x.v;
          lane_elem(sb + 10 * a.Ep, p.ji) = x.w;
        }
        if (f0) lane_elem(sb + 13 * a.Ep, p.jc) = fs[0];
        if (f1) lane_elem(sb + 17 * a.Ep, p.jc) = fs[1];
      }
      if constexpr (LAG) {
#pragma unroll
        for (int h = 0; h < 2; ++h) fs[h] = fmaf(sc.rho, fs[h] - fcmd[h], fcmd[h]);
      }
      quad_substep<LAG>(L, C, sc, x, ml, ma, gl, ga, dl, da);
    }
  }
}

// The reverse sweep.  TRAJ: one sub-step per control step, inputs from the
// trajectory's rows (the first checkpoint for step 0), else from segbuf.  The
// next sub-step's input and the next control step's dL/d traj and throttles are
// loaded one step ahead, so that a lone wave does not wait for them.
template <bool LAG, bool TRAJ>
__global__ void __launch_bounds__(kQuadBlock) __attribute__((amdgpu_waves_per_eu(2)))
k_adj_quad_bwd(const AdjArgs a, const ClassSegs segs) {
  const QuadPlace p = quad_place(segs, a);
  const ClassConst* __restrict__ cc = segs.cc + p.cls;
  const QuadLane L = quad_lane(threadIdx.x);
  const QuadAdjLane LA = quad_adj_lane(p.c);
  QuadThr thr;
  load_quad_thr(cc, p.c, thr);
  QuadThrCols cols;
  load_quad_cols(cc, p.c, cols);
  const int n_f = thr.lag ? thr.n : 0;
  const bool f0 = p.c < n_f, f1 = p.c + 4 < n_f;
  const QuadStep sc = quad_step_const(cc, a.dt);
  QuadAdjConst C;
  load_quad_adj_const(a.derived, a.Ep, p.j4, p.c, C);
  const int S = TRAJ ? 1 : a.substeps;
  auto load_input = [&](int t, int s, QuadState& y) {
    if constexpr (TRAJ) {
      const float* src = t == 0 ? a.ckpt : a.traj + (int64_t)(t - 1) * a.D * a.E;
      quad_load_state(src, a.E, p.oi, p.oc, f0, f1, y);
    } else {
      quad_load_state(a.segbuf + ((int64_t)t * S + s) * a.D * a.Ep, a.Ep, p.ji, p.jc, f0, f1, y);
    }
  };
  auto load_gtraj = [&](int t, QuadLambda& g) {
    const float* gt = a.gtraj + (int64_t)t * a.D * a.E;
    g.p = lane_elem(gt, p.oi);
    g.q = lane_elem(gt + 3 * a.E, p.oc);
    g.v = lane_elem(gt + 7 * a.E, p.oi);
    g.w = lane_elem(gt + 10 * a.E, p.oi);
    g.f[0] = f0 ? lane_elem(gt + 13 * a.E, p.oc) : 0.0f;
    g.f[1] = f1 ? lane_elem(gt + 17 * a.E, p.oc) : 0.0f;
  };
  QuadLambda lam = {0.0f, 0.0f, 0.0f, 0.0f, {0.0f, 0.0f}}, gn;
  QuadTheta th = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
  QuadState yn;
  float an[2];
  load_input(a.T - 1, S - 1, yn);
  load_gtraj(a.T - 1, gn);
  quad_load_throttles(a, p, thr.n, a.T - 1, an);
  for (int t = a.T - 1; t >= 0; --t) {
    const float act[2] = {an[0], an[1]};
    lam.p += gn.p;
    lam.q += gn.q;
    lam.v += gn.v;
    lam.w += gn.w;
    lam.f[0] += gn.f[0];
    lam.f[1] += gn.f[1];
    if (t > 0) {
      load_gtraj(t - 1, gn);
      quad_load_throttles(a, p, thr.n, t - 1, an);
    }
    float fcmd[2], gl, ga, fcb[2] = {0.0f, 0.0f}, gcl = 0.0f, gca = 0.0f, ab[2];
    quad_thrust(thr, act, fcmd);
    quad_wrench(thr, fcmd, gl, ga);
    for (int s = S - 1; s >= 0; --s) {
      const QuadState y = yn;
      if (s > 0)
        load_input(t, s - 1, yn);
      else if (t > 0)
        load_input(t - 1, S - 1, yn);
      quad_substep_vjp<LAG>(L, LA, C, thr, cols, sc, y, fcmd, gl, ga, lam, fcb, gcl, gca, th);
    }
    quad_throttle_vjp(thr, cols, act, fcb, gcl, gca, ab);
    if (p.active) {
      float* gact = a.gact + (int64_t)t * a.n_max * a.E;
      if (p.c < a.n_max) lane_elem(gact, p.oc) = p.c < thr.n ? ab[0] : 0.0f;
      if (p.c + 4 < a.n_max) lane_elem(gact + 4 * a.E, p.oc) = p.c + 4 < thr.n ? ab[1] : 0.0f;
    }
  }
  if (!p.active) return;
  // theta = (M_A(6), D_L(6), D_Q(6), B)
  if (p.c > 0) {
    lane_elem(a.gtheta, p.oi) = th.mal;
    lane_elem(a.gtheta + 3 * a.E, p.oi) = th.maa;
    lane_elem(a.gtheta + 6 * a.E, p.oi) = th.dll;
    lane_elem(a.gtheta + 9 * a.E, p.oi) = th.dla;
    lane_elem(a.gtheta + 12 * a.E, p.oi) = th.dql;
    lane_elem(a.gtheta + 15 * a.E, p.oi) = th.dqa;
  } else {
    lane_elem(a.gtheta + 18 * a.E, p.c4) = fmaf(-segs.zb[p.cls], th.hz, -th.wmb);
  }
  if (a.gx0)
    quad_store_caller(a.gx0, a, p, f0, f1, lam.p, lam.q, lam.v, lam.w, lam.f[0], lam.f[1]);
}

// 32-bit offsets of a state's rows
static bool quad_fits(const AdjArgs& a) { return a.Ep <= kQuadMaxEnvs && a.E <= kQuadMaxEnvs; }

hipError_t launch_adj_quad_fwd(const ClassSegs& q, const AdjArgs& a, bool lag, hipStream_t s) {
  if (!quad_fits(a)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)q.blk_end[q.n - 1]);
  if (lag)
    hipLaunchKernelGGL((k_adj_quad_fwd<true>), grid, dim3(kQuadBlock), 0, s, a, q);
  else
    hipLaunchKernelGGL((k_adj_quad_fwd<false>), grid, dim3(kQuadBlock), 0, s, a, q);
  return hipGetLastError();
}

hipError_t launch_adj_quad_recompute(const ClassSegs& q, const AdjArgs& a, bool lag,
                                     hipStream_t s) {
  const int ny = (a.T + a.ckpt_every - 1) / a.ckpt_every;
  if (!quad_fits(a) || ny > 65535) return hipErrorInvalidValue;
  const dim3 grid((unsigned)q.blk_end[q.n - 1], (unsigned)ny);
  if (lag)
    hipLaunchKernelGGL((k_adj_quad_recompute<true>), grid, dim3(kQuadBlock), 0, s, a, q);
  else
    hipLaunchKernelGGL((k_adj_quad_recompute<false>), grid, dim3(kQuadBlock), 0, s, a, q);
  return hipGetLastError();
}

hipError_t launch_adj_quad_bwd(const ClassSegs& q, const AdjArgs& a, bool lag, hipStream_t s) {
  if (!quad_fits(a)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)q.blk_end[q.n - 1]), block(kQuadBlock);
  const bool traj = a.recomputed == 2;
  if (lag && traj)
    hipLaunchKernelGGL((k_adj_quad_bwd<true, true>), grid, block, 0, s, a, q);
  else if (lag)
    hipLaunchKernelGGL((k_adj_quad_bwd<true, false>), grid, block, 0, s, a, q);
  else if (traj)
    hipLaunchKernelGGL((k_adj_quad_bwd<false, true>), grid, block, 0, s, a, q);
  else
    hipLaunchKernelGGL((k_adj_quad_bwd<false, false>), grid, block, 0, s, a, q);
  return hipGetLastError();
}

}  // namespace mg
