// kernels_adjoint_quad.hip -- the adjoint's recomputation and reverse sweep with
// one env per quad of lanes and all classes in one launch (fossen_quad_adjoint.h),
// for sims too small to fill the GPU with one env per lane (their forward is
// k_roll_quad): a launch then lasts as long as one env's chain of sub-steps, at
// 2.1 ns an instruction for a lone wave.  Results are bitwise those of
// kernels_adjoint.hip.  16 control steps, one env per lane and here, forward /
// backward: 1000 envs without lag, one sub-step 27.6 / 55.7 -> 12.1 / 19.7 us; 8192
// 28.8 / 56.6 -> 14.0 / 23.0; 16 384 28.0 / 57.9 -> 17.0 / 33.1; with lag and four
// sub-steps, 1000 envs 72 / 244 -> 33 / 87, 8192 74 / 251 -> 37 / 102, 16 384
// 74 / 252 -> 40 / 149.
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
  int n;                // the class's thrusters
  QuadPair jf, of, oa;  // lag states in internal and caller rows, throttles
};

// b: the block of kQuadEnvs envs (one past the last in the surplus half of a
// paired sweep's last block)
__device__ __forceinline__ QuadPlace quad_place(const ClassSegs& segs, const AdjArgs& a, int b) {
  QuadPlace p;
  const int lane = threadIdx.x & (kQuadBlock - 1);
  const QuadEnv e = quad_env(a, segs, b, lane);
  const int k = e.cls;
  p.cls = k;
  p.c = lane & 3;
  const int ci = p.c > 1 ? p.c - 1 : 0;
  p.active = e.active;
  p.j4 = e.j * 4u;
  const int64_t col = p.active ? (a.perm ? (int64_t)lane_elem(a.perm, p.j4) : (int64_t)e.j) : 0;
  p.active = p.active && MG_CHECK(a, col >= 0 && col < a.dbg.cols, kDbgColumn);
  p.c4 = p.active ? (uint32_t)col * 4u : 0u;
  const uint32_t s4 = (uint32_t)a.Ep * 4u, e4 = (uint32_t)a.E * 4u;
  p.ji = p.j4 + (uint32_t)ci * s4;
  p.jc = p.j4 + (uint32_t)p.c * s4;
  p.oi = p.c4 + (uint32_t)ci * e4;
  p.oc = p.c4 + (uint32_t)p.c * e4;
  p.n = segs.cc[k].n_thr;
  const int n_f = segs.cc[k].lag ? p.n : 0;
  p.jf = quad_pair(p.c, n_f, p.j4, s4);
  p.of = quad_pair(p.c, n_f, p.c4, e4);
  p.oa = quad_pair(p.c, p.n, p.c4, e4);
  return p;
}

// One state's rows, row stride ld floats; lane offsets vi (3-vectors), vc, f (lag
// states, to be masked).
template <bool LAG>
__device__ __forceinline__ void quad_load_state(const float* rows, int64_t ld, uint32_t vi,
                                                uint32_t vc, const QuadPair& f, QuadState& x) {
  x.q = lane_elem(rows + 3 * ld, vc);
  x.v = lane_elem(rows + 7 * ld, vi);
  x.w = lane_elem(rows + 10 * ld, vi);
  x.f[0] = x.f[1] = 0.0f;
  if constexpr (LAG) quad_load_pair(f, rows + 13 * ld, x.f);
}

// A caller state [D][E]: lag states past the class's are zeros.
template <bool LAG>
__device__ __forceinline__ void quad_store_caller(float* rows, const AdjArgs& a,
                                                  const QuadPlace& p, float xp, float xq, float xv,
                                                  float xw, const float (&f)[2]) {
  lane_elem(rows + 3 * a.E, p.oc) = xq;
  if (p.c > 0) {
    lane_elem(rows, p.oi) = xp;
    lane_elem(rows + 7 * a.E, p.oi) = xv;
    lane_elem(rows + 10 * a.E, p.oi) = xw;
  }
  if constexpr (LAG) {
    if (13 + p.c < a.D) lane_elem(rows + 13 * a.E, p.oc) = f[0];
    if (17 + p.c < a.D) lane_elem(rows + 17 * a.E, p.oc) = f[1];
  }
}

__device__ __forceinline__ void quad_load_throttles(const AdjArgs& a, const QuadPlace& p, int t,
                                                    float (&act)[2]) {
  quad_load_pair(p.oa, a.actions + (int64_t)t * a.n_max * a.E, act);
}

}  // namespace

// Every segment's sub-step inputs at once (blockIdx.y = segment) into the
// whole-rollout segbuf.  Position rows are left out: the sweep reads none.
template <bool LAG>
__global__ void __launch_bounds__(kQuadBlock) k_adj_quad_recompute(const AdjArgs a,
                                                                   const ClassSegs segs) {
  const QuadPlace p = quad_place(segs, a, blockIdx.x);
  const ClassConst* __restrict__ cc = segs.cc + p.cls;
  const QuadLane L = quad_lane(threadIdx.x);
  QuadThr th;
  load_quad_thr(cc, p.c, th);
  const int seg = blockIdx.y;
  const int t0 = seg * a.ckpt_every, t1 = min(a.T, t0 + a.ckpt_every);
  const float* src = a.ckpt + (int64_t)seg * a.D * a.E;
  QuadState x;
  x.p = 0.0f;
  quad_load_state<LAG>(src, a.E, p.oi, p.oc, p.of, x);
  const QuadStep sc = quad_step_const(cc, a.dt);
  QuadConst C;
  QuadMass M;
  load_quad_const(a.derived, a.Ep, p.j4, p.c, sc.h2, C, M);
  if constexpr (LAG) quad_mask_pair(p.of, x.f);
  for (int t = t0; t < t1; ++t) {
    float act[2], fcmd[2], gl, ga, dl, da, ml, ma;
    quad_load_throttles(a, p, t, act);
    quad_mask_pair(p.oa, act);
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
        if constexpr (LAG) quad_store_pair(p.jf, sb + 13 * a.Ep, fs);
      }
      if constexpr (LAG) {
#pragma unroll
        for (int h = 0; h < 2; ++h) fs[h] = fmaf(sc.rho, fs[h] - fcmd[h], fcmd[h]);
      }
      quad_substep<LAG>(L, C, sc, x, ml, ma, gl, ga, dl, da);
    }
  }
}

// The loads of the reverse sweep.  TRAJ: one sub-step per control step, inputs
// from the trajectory's rows (the first checkpoint for step 0), else from segbuf.
template <bool LAG, bool TRAJ>
__device__ __forceinline__ void quad_load_input(const AdjArgs& a, const QuadPlace& p, int S, int t,
                                                int s, QuadState& y) {
  if constexpr (TRAJ) {
    const float* src = t == 0 ? a.ckpt : a.traj + (int64_t)(t - 1) * a.D * a.E;
    quad_load_state<LAG>(src, a.E, p.oi, p.oc, p.of, y);
  } else {
    quad_load_state<LAG>(a.segbuf + ((int64_t)t * S + s) * a.D * a.Ep, a.Ep, p.ji, p.jc, p.jf, y);
  }
}
__device__ __forceinline__ void quad_load_gtraj(const AdjArgs& a, const QuadPlace& p, int t,
                                                QuadLambda& g) {
  const float* gt = a.gtraj + (int64_t)t * a.D * a.E;
  g.p = lane_elem(gt, p.oi);
  g.q = lane_elem(gt + 3 * a.E, p.oc);
  g.v = lane_elem(gt + 7 * a.E, p.oi);
  g.w = lane_elem(gt + 10 * a.E, p.oi);
}
template <bool LAG>
__device__ __forceinline__ void quad_load_gtraj_f(const AdjArgs& a, const QuadPlace& p, int t,
                                                  float (&g)[2]) {
  g[0] = g[1] = 0.0f;
  if constexpr (LAG) quad_load_pair(p.of, a.gtraj + ((int64_t)t * a.D + 13) * a.E, g);
}
__device__ __forceinline__ void quad_store_gact(const AdjArgs& a, const QuadPlace& p, int t,
                                                float (&ab)[2]) {
  float* gact = a.gact + (int64_t)t * a.n_max * a.E;
  quad_mask_pair(p.oa, ab);
  if (p.c < a.n_max) lane_elem(gact, p.oc) = ab[0];
  if (p.c + 4 < a.n_max) lane_elem(gact + 4 * a.E, p.oc) = ab[1];
}
// theta = (M_A(6), D_L(6), D_Q(6), B)
__device__ __forceinline__ void quad_store_theta(const AdjArgs& a, const QuadPlace& p, float zb,
                                                 const QuadTheta& th) {
  if (p.c > 0) {
    lane_elem(a.gtheta, p.oi) = th.mal;
    lane_elem(a.gtheta + 3 * a.E, p.oi) = th.maa;
    lane_elem(a.gtheta + 6 * a.E, p.oi) = th.dll;
    lane_elem(a.gtheta + 9 * a.E, p.oi) = th.dla;
    lane_elem(a.gtheta + 12 * a.E, p.oi) = th.dql;
    lane_elem(a.gtheta + 15 * a.E, p.oi) = th.dqa;
  } else {
    lane_elem(a.gtheta + 18 * a.E, p.c4) = fmaf(-zb, th.hz, -th.wmb);
  }
}

// The reverse sweep in one wave.  The next sub-step's input and the next control
// step's dL/d traj and throttles are loaded one step ahead, so that a lone wave
// does not wait for them.
template <bool LAG, bool TRAJ>
__global__ void __launch_bounds__(kQuadBlock) __attribute__((amdgpu_waves_per_eu(2)))
k_adj_quad_bwd(const AdjArgs a, const ClassSegs segs) {
  const QuadPlace p = quad_place(segs, a, blockIdx.x);
  const ClassConst* __restrict__ cc = segs.cc + p.cls;
  const QuadLane L = quad_lane(threadIdx.x);
  const QuadAdjLane LA = quad_adj_lane(p.c);
  QuadThr thr;
  load_quad_thr(cc, p.c, thr);
  QuadThrCols cols;
  load_quad_cols(cc, p.c, cols);
  const QuadStep sc = quad_step_const(cc, a.dt);
  QuadAdjConst C;
  load_quad_adj_const(a.derived, a.Ep, p.j4, p.c, C);
  const int S = TRAJ ? 1 : a.substeps;
  QuadLambda lam = {0.0f, 0.0f, 0.0f, 0.0f}, gn;
  QuadThrBar tb = {{0.0f, 0.0f}, {0.0f, 0.0f}, 0.0f, 0.0f};
  QuadTheta th = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
  QuadState yn;
  float an[2], fn[2];
  quad_load_input<LAG, TRAJ>(a, p, S, a.T - 1, S - 1, yn);
  quad_load_gtraj(a, p, a.T - 1, gn);
  quad_load_gtraj_f<LAG>(a, p, a.T - 1, fn);
  quad_load_throttles(a, p, a.T - 1, an);
  for (int t = a.T - 1; t >= 0; --t) {
    float act[2] = {an[0], an[1]};
    quad_mask_pair(p.oa, act);
    if constexpr (LAG) quad_mask_pair(p.of, fn);
    lam.p += gn.p;
    lam.q += gn.q;
    lam.v += gn.v;
    lam.w += gn.w;
    tb.lam[0] += fn[0];
    tb.lam[1] += fn[1];
    if (t > 0) {
      quad_load_gtraj(a, p, t - 1, gn);
      quad_load_gtraj_f<LAG>(a, p, t - 1, fn);
      quad_load_throttles(a, p, t - 1, an);
    }
    float fcmd[2], gl, ga, ab[2];
    quad_thrust(thr, act, fcmd);
    quad_wrench(thr, fcmd, gl, ga);
    tb.fcb[0] = tb.fcb[1] = tb.gcl = tb.gca = 0.0f;
    for (int s = S - 1; s >= 0; --s) {
      QuadState y = yn;
      if constexpr (LAG) quad_mask_pair(p.jf, y.f);
      if (s > 0)
        quad_load_input<LAG, TRAJ>(a, p, S, t, s - 1, yn);
      else if (t > 0)
        quad_load_input<LAG, TRAJ>(a, p, S, t - 1, S - 1, yn);
      QuadStages st;
      QuadStageOut o[4];
      quad_stages<LAG>(L, C, thr, sc, y, fcmd, gl, ga, st);
      quad_substep_vjp(
          p.c, LA, C, sc, st.qo, st.inv, [&](int i) { return st.s[i]; },
          [&](int i, const QuadStageOut& v) {
            o[i] = v;
            quad_stage_theta(st.t[i], v, th);
          },
          lam);
      quad_thrusters_vjp<LAG>(thr, cols, sc, o, tb);
    }
    quad_throttle_vjp(thr, cols, act, tb, ab);
    if (p.active) quad_store_gact(a, p, t, ab);
  }
  if (!p.active) return;
  quad_store_theta(a, p, segs.zb[p.cls], th);
  quad_mask_pair(p.of, tb.lam);
  if (a.gx0)
    quad_store_caller<LAG>(a.gx0, a, p, lam.p, lam.q, lam.v, lam.w, tb.lam);
}

// The reverse sweep in three waves per 16 envs.  Only the chain of state adjoints
// is serial over the sub-steps; the stages' forward values ahead of it and the
// parameter and thruster adjoints behind it are not.  In phase h wave 0 (the
// chain) reverses sub-step N - h while wave 1 forms the stages of sub-step
// N - 1 - h and wave 2 folds what sub-step N + 1 - h left for the parameters and
// thrusters, all through LDS; one barrier per phase, N + 2 phases for every wave
// alike.  The values and their order are those of the one-wave sweep, bitwise.
//
// LDS holds float4 columns of 64 lanes: the chain's input (16 values of each
// stage, q and 1/|q|) twice, what the parameters read of the stages (5 of each)
// three times, and of the chain (4 of each) twice: 57 KiB, two blocks to a CU.
// 445 instructions in wave 0's phase, of them 345 VALU for a sub-step, against 710-980
// of the one-wave sweep (660-740 VALU), 370-450 in wave 1's, 200-300 in wave 2's.
constexpr int kTrioIn = 17, kTrioTheta = 5, kTrioOut = 4;   // columns
constexpr int kTrioColumns = 2 * kTrioIn + 3 * kTrioTheta + 2 * kTrioOut;

// PAIR: two groups of 16 envs to a block of eight waves, one block to a CU, for
// launches of more groups than CUs.  A block's waves go to the CU's four SIMDs in
// turn, so waves 0 and 1, the two chains, have a SIMD each, which waves 4 and 5
// leave to them (they only keep the barriers), and each of the other two SIMDs
// takes one group's waves 1 and 2 of above.  As two blocks of three waves a chain
// shares its SIMD (8192 envs as above: 29.1 against 23.5 us without lag, 129
// against 103 with; in one wave 33.8 and 148).
template <bool LAG, bool TRAJ, bool PAIR>
__global__ void __launch_bounds__((PAIR ? 8 : 3) * kQuadBlock)
    __attribute__((amdgpu_waves_per_eu(2)))
k_adj_quad_bwd_trio(const AdjArgs a, const ClassSegs segs) {
  __shared__ float4 lds_all[PAIR ? 2 : 1][kTrioColumns][kQuadBlock];
  const int lane = threadIdx.x & (kQuadBlock - 1);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kQuadBlock);
  const int group = PAIR ? wv & 1 : 0;
  // 0 chain, 1 stages, 2 fold, 3 none
  const int wave = PAIR ? (wv < 2 ? 0 : (wv < 4 ? 1 : (wv < 6 ? 3 : 2))) : wv;
  auto& lds = lds_all[group];
  auto col_in = [&](int buf, int i) -> float4& { return lds[buf * kTrioIn + i][lane]; };
  auto col_out = [&](int buf, int i) -> float4& {
    return lds[2 * kTrioIn + buf * kTrioOut + i][lane];
  };
  auto col_theta = [&](int buf, int i) -> float4& {
    return lds[2 * (kTrioIn + kTrioOut) + buf * kTrioTheta + i][lane];
  };
  const QuadPlace p = quad_place(segs, a, PAIR ? 2 * (int)blockIdx.x + group : (int)blockIdx.x);
  const ClassConst* __restrict__ cc = segs.cc + p.cls;
  const QuadStep sc = quad_step_const(cc, a.dt);
  QuadAdjConst C;
  load_quad_adj_const(a.derived, a.Ep, p.j4, p.c, C);
  const int S = TRAJ ? 1 : a.substeps, N = a.T * S;
  if (wave == 3) {
    for (int h = 0; h < N + 2; ++h) lds_barrier();
    return;
  }
  if (wave == 0) {
    const QuadAdjLane LA = quad_adj_lane(p.c);
    QuadLambda lam = {0.0f, 0.0f, 0.0f, 0.0f}, gn;
    quad_load_gtraj(a, p, a.T - 1, gn);
    int t = a.T - 1, s = S - 1;
    for (int h = 0; h < N + 2; ++h) {
      if (h > 0 && h <= N) {
        const int buf = (N - h) & 1;
        if (s == S - 1) {
          lam.p += gn.p;
          lam.q += gn.q;
          lam.v += gn.v;
          lam.w += gn.w;
          if (t > 0) quad_load_gtraj(a, p, t - 1, gn);
        }
        // all of it at once, ahead of the stores to LDS below
        float4 u[17];
#pragma unroll
        for (int i = 16; i >= 0; --i) u[i] = col_in(buf, i);
        quad_substep_vjp(
            p.c, LA, C, sc, u[16].x, u[16].y,
            [&](int i) {
              const float4 u0 = u[4 * i], u1 = u[4 * i + 1], u2 = u[4 * i + 2], u3 = u[4 * i + 3];
              return QuadStage{u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w,
                               u2.x, u2.y, u2.z, u2.w, u3.x, u3.y, u3.z, u3.w};
            },
            [&](int i, const QuadStageOut& o) {
              col_out(buf, i) = make_float4(o.f, o.m, o.ab, o.bb);
            },
            lam);
        if (--s < 0) {
          s = S - 1;
          --t;
        }
      }
      lds_barrier();
    }
    if (p.active && a.gx0) {
      lane_elem(a.gx0 + 3 * a.E, p.oc) = lam.q;
      if (p.c > 0) {
        lane_elem(a.gx0, p.oi) = lam.p;
        lane_elem(a.gx0 + 7 * a.E, p.oi) = lam.v;
        lane_elem(a.gx0 + 10 * a.E, p.oi) = lam.w;
      }
    }
    return;
  }
  QuadThr thr;
  load_quad_thr(cc, p.c, thr);
  if (wave == 1) {
    const QuadLane L = quad_lane(lane);
    QuadState yn;
    float an[2], fcmd[2], gl = 0.0f, ga = 0.0f;
    int t = a.T - 1, s = S - 1, ring = 0;
    quad_load_input<LAG, TRAJ>(a, p, S, t, s, yn);
    quad_load_throttles(a, p, t, an);
    for (int h = 0; h < N + 2; ++h) {
      if (h < N) {
        const int buf = (N - 1 - h) & 1;
        if (s == S - 1) {
          quad_mask_pair(p.oa, an);
          quad_thrust(thr, an, fcmd);
          quad_wrench(thr, fcmd, gl, ga);
          if (t > 0) quad_load_throttles(a, p, t - 1, an);
        }
        QuadState y = yn;
        if constexpr (LAG) quad_mask_pair(p.jf, y.f);
        if (--s < 0) {
          s = S - 1;
          --t;
        }
        if (t >= 0) quad_load_input<LAG, TRAJ>(a, p, S, t, s, yn);
        QuadStages st;
        quad_stages<LAG>(L, C, thr, sc, y, fcmd, gl, ga, st);
        float v[20];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const QuadStage& g = st.s[i];
          col_in(buf, 4 * i) = make_float4(g.q, g.qw, g.q1, g.q2);
          col_in(buf, 4 * i + 1) = make_float4(g.v1, g.v2, g.w, g.w1);
          col_in(buf, 4 * i + 2) = make_float4(g.w2, g.t, g.a1, g.a2);
          col_in(buf, 4 * i + 3) = make_float4(g.b1, g.b2, g.el, g.ea);
          v[5 * i] = st.t[i].v;
          v[5 * i + 1] = st.t[i].w;
          v[5 * i + 2] = st.t[i].k;
          v[5 * i + 3] = st.t[i].nl;
          v[5 * i + 4] = st.t[i].na;
        }
        col_in(buf, 16) = make_float4(st.qo, st.inv, 0.0f, 0.0f);
#pragma unroll
        for (int i = 0; i < 5; ++i)
          col_theta(ring, i) = make_float4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
        ring = ring == 2 ? 0 : ring + 1;
      }
      lds_barrier();
    }
    return;
  }
  QuadThrCols cols;
  load_quad_cols(cc, p.c, cols);
  QuadThrBar tb = {{0.0f, 0.0f}, {0.0f, 0.0f}, 0.0f, 0.0f};
  QuadTheta th = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
  float an[2], fn[2], act[2] = {0.0f, 0.0f};
  int t = a.T - 1, s = S - 1, ring = 0;
  quad_load_throttles(a, p, t, an);
  quad_load_gtraj_f<LAG>(a, p, t, fn);
  for (int h = 0; h < N + 2; ++h) {
    if (h > 1) {
      const int buf = (N + 1 - h) & 1;
      float v[20];
#pragma unroll
      for (int i = 0; i < 5; ++i) {
        const float4 u = col_theta(ring, i);
        v[4 * i] = u.x;
        v[4 * i + 1] = u.y;
        v[4 * i + 2] = u.z;
        v[4 * i + 3] = u.w;
      }
      ring = ring == 2 ? 0 : ring + 1;
      if (s == S - 1) {
        act[0] = an[0];
        act[1] = an[1];
        quad_mask_pair(p.oa, act);
        if constexpr (LAG) quad_mask_pair(p.of, fn);
        tb.lam[0] += fn[0];
        tb.lam[1] += fn[1];
        tb.fcb[0] = tb.fcb[1] = tb.gcl = tb.gca = 0.0f;
        if (t > 0) {
          quad_load_throttles(a, p, t - 1, an);
          quad_load_gtraj_f<LAG>(a, p, t - 1, fn);
        }
      }
      QuadStageOut o[4];
#pragma unroll
      for (int i = 3; i >= 0; --i) {
        const float4 u = col_out(buf, i);
        o[i] = {u.x, u.y, u.z, u.w};
        quad_stage_theta({v[5 * i], v[5 * i + 1], v[5 * i + 2], v[5 * i + 3], v[5 * i + 4]}, o[i],
                         th);
      }
      quad_thrusters_vjp<LAG>(thr, cols, sc, o, tb);
      if (s == 0) {
        float ab[2];
        quad_throttle_vjp(thr, cols, act, tb, ab);
        if (p.active) quad_store_gact(a, p, t, ab);
      }
      if (--s < 0) {
        s = S - 1;
        --t;
      }
    }
    lds_barrier();
  }
  if (!p.active) return;
  quad_store_theta(a, p, segs.zb[p.cls], th);
  if constexpr (LAG) {
    quad_mask_pair(p.of, tb.lam);
    if (a.gx0 && 13 + p.c < a.D) lane_elem(a.gx0 + 13 * a.E, p.oc) = tb.lam[0];
    if (a.gx0 && 17 + p.c < a.D) lane_elem(a.gx0 + 17 * a.E, p.oc) = tb.lam[1];
  }
}

// 32-bit offsets of a state's rows
static bool quad_fits(const AdjArgs& a) { return a.Ep <= kQuadMaxEnvs && a.E <= kQuadMaxEnvs; }

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
  const int nblk = q.blk_end[q.n - 1];
  const bool traj = a.recomputed == 2;
#define MG_LAUNCH(grid, block, kernel, ...)                                                       \
  do {                                                                                            \
    const dim3 g((unsigned)(grid)), b(block);                                                     \
    if (lag && traj)                                                                              \
      hipLaunchKernelGGL((kernel<true, true __VA_ARGS__>), g, b, 0, s, a, q);                     \
    else if (lag)                                                                                 \
      hipLaunchKernelGGL((kernel<true, false __VA_ARGS__>), g, b, 0, s, a, q);                    \
    else if (traj)                                                                                \
      hipLaunchKernelGGL((kernel<false, true __VA_ARGS__>), g, b, 0, s, a, q);                    \
    else                                                                                          \
      hipLaunchKernelGGL((kernel<false, false __VA_ARGS__>), g, b, 0, s, a, q);                   \
  } while (0)
  // three waves per group of 16 envs while a CU holds at most two groups (and
  // the phases fit an int), else one wave
  const bool phases = (int64_t)a.T * a.substeps < INT32_MAX - 2;
  if (phases && nblk <= a.n_cu)
    MG_LAUNCH(nblk, 3 * kQuadBlock, k_adj_quad_bwd_trio, , false);
  else if (phases && nblk <= 2 * a.n_cu)
    MG_LAUNCH((nblk + 1) / 2, 8 * kQuadBlock, k_adj_quad_bwd_trio, , true);
  else
    MG_LAUNCH(nblk, kQuadBlock, k_adj_quad_bwd, );
#undef MG_LAUNCH
  return hipGetLastError();
}

}  // namespace mg
