"""GPU checks of the kernels that take all classes in one launch: those with one env over a
quad of lanes (sims of at most one wave per SIMD) against the ones with one env per lane, the
same envs inside a batch too large for the quad kernels, bitwise, at the edges of a wave's 16
envs and of the range; and a rollout in one launch against its steps."""
import sys
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

from tests.gpu_util import TOL_ONE_STEP, dev, host, rel_err, say                                  # noqa: E402
from workloads import (BLUEROV2, BLUEROV2_HEAVY, actions, param_multipliers,   # noqa: E402
                       random_states, vehicle_variant)

pytestmark = pytest.mark.gpu

BIG = 20000       # more than one quad wave per SIMD of 256 CUs (16384 envs)
LAG_HEAVY = vehicle_variant(BLUEROV2_HEAVY, thr_map=1, thr_tau=0.05)
LAG_BLUE = vehicle_variant(BLUEROV2, thr_map=1, thr_tau=0.05)
THREE = dict(BLUEROV2, thr_pos=BLUEROV2["thr_pos"][:3], thr_dir=BLUEROV2["thr_dir"][:3])
FLEETS = {"heavy": [LAG_HEAVY], "bluerov2": [BLUEROV2], "three": [THREE],
          "mixed": [LAG_BLUE, LAG_HEAVY], "plain_mixed": [BLUEROV2, BLUEROV2_HEAVY],
          "lag_and_not": [LAG_HEAVY, BLUEROV2]}


@pytest.fixture(scope="module")
def mgmod():
    from paper_2410_14117_amd import mg
    mg.lib()
    return mg


def _inputs(classes, E, T, seed):
    lagged = max([len(v["thr_pos"]) for v in classes if v["thr_tau"] > 0] or [0])
    n_max = max(len(v["thr_pos"]) for v in classes)
    cls = np.random.default_rng(seed).integers(0, len(classes), E).astype(np.int32)
    x0 = random_states(E, 13 + lagged, seed + 1)
    for k, v in enumerate(classes):
        x0[13 + (len(v["thr_pos"]) if v["thr_tau"] > 0 else 0):, cls == k] = 0
    return cls, x0, 1.2 * actions(T, n_max, E, seed + 2), param_multipliers(E, 0.2, seed + 3)


def _run(mg, classes, cls, x0, act, mult, S, mode, E):
    sim = mg.Sim(classes, E, 0.005, S, env_class=cls[:E])
    sim.reset(state=dev(x0[:, :E]), param_mult=dev(mult[:, :E]))
    T = act.shape[0]
    traj = torch.full((T, x0.shape[0], E), -1.0, device="cuda")
    stats = torch.empty((T, 4), dtype=torch.float64, device="cuda")
    fn = sim.rollout if mode == "rollout" else sim.step
    fn(dev(act[:, :, :E]), traj=traj, stats=stats)
    out = host(traj), host(stats), host(sim.get_state()), host(sim.get_flags())
    sim.close()
    return out


@pytest.mark.parametrize("fleet,S,T,mode,sizes", [
    ("heavy", 4, 3, "step", (1, 15, 16, 17, 16384)),
    ("bluerov2", 1, 130, "rollout", (33,)),     # more than one piece of the statistics
    ("three", 2, 3, "step", (49,)),
    ("mixed", 4, 5, "rollout", (2, 1001)),
    ("lag_and_not", 2, 4, "step", (1001,)),
])
def test_quad_step_equals_one_env_per_lane(mgmod, fleet, S, T, mode, sizes):
    classes = FLEETS[fleet]
    cls, x0, act, mult = _inputs(classes, BIG, T, 11)
    say("quad step", fleet, S, T, mode)
    big = _run(mgmod, classes, cls, x0, act, mult, S, mode, BIG)
    for E in sizes:
        say("  envs", E)
        traj, stats, xT, flags = _run(mgmod, classes, cls, x0, act, mult, S, mode, E)
        np.testing.assert_array_equal(traj, big[0][:, :, :E])
        np.testing.assert_array_equal(xT, big[2][:, :E])
        assert not flags.any() and not stats[:, 3].any()
        # FP64 sums of the same FP32 positions in another order
        d = np.sqrt((traj[:, :3].astype(np.float64) ** 2).sum(1))
        np.testing.assert_allclose(stats[:, 0], d.sum(1), rtol=1e-12)
        np.testing.assert_allclose(stats[:, 1], d.max(1), rtol=1e-12)


@pytest.mark.parametrize("mode", ["step", "rollout"])
def test_quad_freeze_equals_one_env_per_lane(mgmod, mode):
    """An env whose throttles turn NaN part-way, in a launch of several control steps and in a
    rollout: the same frozen state, flags, counts and later trajectory rows either way."""
    classes, T = FLEETS["mixed"], 6
    cls, x0, act, mult = _inputs(classes, BIG, T, 21)
    act[2, 1, 5] = np.nan
    act[0, 0, 18] = np.nan
    say("quad freeze", mode)
    big = _run(mgmod, classes, cls, x0, act, mult, 2, mode, BIG)
    traj, stats, xT, flags = _run(mgmod, classes, cls, x0, act, mult, 2, mode, 40)
    np.testing.assert_array_equal(xT, big[2][:, :40])
    np.testing.assert_array_equal(flags, big[3][:40])
    assert list(np.flatnonzero(flags)) == [5, 18]
    np.testing.assert_array_equal(traj, big[0][:, :, :40])
    assert list(stats[:, 3]) == [1, 1, 2, 2, 2, 2]


def _grads(mg, classes, cls, x0, act, mult, g, S, K, mode, E):
    sim = mg.Sim(classes, E, 0.005, S, env_class=cls[:E])
    sim.reset(state=dev(x0[:, :E]), param_mult=dev(mult[:, :E]))
    a = dev(act[:, :, :E])
    traj = torch.full((act.shape[0], x0.shape[0], E), -1.0, device="cuda")
    ckpt, _ = sim.adj_forward(a, K, traj=traj)
    out = sim.adj_backward(ckpt, a, K, dev(g[:, :, :E]), traj=None if mode == "ckpt" else traj,
                           noalloc=mode == "noalloc")
    out = [host(v) for v in (ckpt, traj) + out] + [host(sim.get_state())]
    sim.close()
    return out


@pytest.mark.parametrize("fleet,S,T,K,mode,sizes", [
    ("heavy", 3, 5, 2, "ckpt", (1, 17, 4096, 4097, 8192, 8193, 16384)),
    ("heavy", 2, 4, 4, "noalloc", (33,)),       # one segment, recomputed ahead of the sweep
    ("bluerov2", 1, 7, 3, "traj", (16, 1001, 5001, 9000)),
    ("three", 1, 1, 2, "ckpt", (49, 5000)),     # a single sub-step
    ("mixed", 2, 5, 2, "ckpt", (2, 1001, 4100)),
    ("lag_and_not", 1, 5, 2, "traj", (1001, 6000, 10000)),
])
def test_quad_adjoint_equals_one_env_per_lane(mgmod, fleet, S, T, K, mode, sizes):
    """Checkpoints, trajectory, final state and every gradient, bitwise; on 256 compute units
    the sweep takes three waves per 16 envs up to 4096 envs, blocks of two such groups up to
    8192 and one wave beyond."""
    classes = FLEETS[fleet]
    cls, x0, act, mult = _inputs(classes, BIG, T, 31)
    g = np.random.default_rng(35).standard_normal((T,) + x0.shape).astype(np.float32)
    say("quad adjoint", fleet, S, T, K, mode)
    big = _grads(mgmod, classes, cls, x0, act, mult, g, S, K, "ckpt", BIG)
    for E in sizes:
        say("  envs", E)
        got = _grads(mgmod, classes, cls, x0, act, mult, g, S, K, mode, E)
        for name, u, w in zip(("ckpt", "traj", "gact", "gtheta", "gx0", "state"), got, big):
            np.testing.assert_array_equal(u, w[..., :E], err_msg=name)


@pytest.mark.parametrize("fleet,S,T,sizes", [
    ("heavy", 4, 3, (1, 17, 16384)),
    ("bluerov2", 1, 5, (33,)),
    ("three", 2, 3, (49,)),
    ("lag_and_not", 3, 4, (2, 1001)),
])
def test_split_of_all_classes_in_one_launch(mgmod, oracle, fleet, S, T, sizes):
    """The split scheme with one env per lane and one per quad of lanes: bitwise equal over two
    calls (the second from carried accelerations), and within the one-step tolerance of the
    oracle for each class's own thrusters."""
    classes = [dict(v, added_mass=[0.4 * m for m in v["added_mass"]]) for v in FLEETS[fleet]]
    cls, x0, act, mult = _inputs(classes, BIG, 2 * T, 41)
    say("split", fleet, S, T)

    def run(E):
        sim = mgmod.Sim(classes, E, 0.005, S, env_class=cls[:E])
        sim.reset(state=dev(x0[:, :E]), param_mult=dev(mult[:, :E]))
        traj = torch.full((2 * T, x0.shape[0], E), -1.0, device="cuda")
        sim.step_split(dev(act[:T, :, :E]), traj=traj[:T])
        sim.step_split(dev(act[T:, :, :E]), traj=traj[T:])
        out = host(traj), host(sim.get_state())
        sim.close()
        return out

    big = run(BIG)
    for E in sizes:
        say("  envs", E)
        for u, w in zip(run(E), big):
            np.testing.assert_array_equal(u, w[..., :E])
    sub = np.r_[0:8, BIG - 5:BIG]
    ref = oracle.split_rollout(classes, x0[:, sub], act[:1][:, :, sub], S, 0.005,
                               env_class=cls[sub], mult=mult[:, sub], want_traj=True)
    assert rel_err(big[0][0][:, sub], ref["traj"][0]) <= TOL_ONE_STEP


@pytest.mark.parametrize("fleet,E", [("heavy", 16385), ("mixed", 20000), ("bluerov2", 16640),
                                     ("lag_and_not", 20000)])
def test_rollout_of_all_classes_in_one_launch(mgmod, fleet, E):
    """One env per lane: a rollout equals as many single steps (of the same classes one at a
    time if the sim has one class), bitwise, with envs that go non-finite part-way, at the
    first and the last control step, and one that is not steppable from the start."""
    classes, T, S = FLEETS[fleet], 4, 2
    cls, x0, act, mult = _inputs(classes, E, T, 51)
    act[0, 0, 7] = act[1, 1, 100] = act[T - 1, 0, E - 1] = np.nan
    mult[4:7, 300] = -9.0          # mass matrix not positive definite
    say("rollout in one launch", fleet, E)
    out = []
    for mode in ("rollout", "step"):
        sim = mgmod.Sim(classes, E, 0.005, S, env_class=cls)
        sim.reset(state=dev(x0), param_mult=dev(mult))
        traj = torch.full((T, x0.shape[0], E), -1.0, device="cuda")
        stats = torch.empty((T, 4), dtype=torch.float64, device="cuda")
        if mode == "rollout":
            sim.rollout(dev(act), traj=traj, stats=stats)
        else:
            for t in range(T):
                sim.step(dev(act[t:t + 1]), traj=traj[t:t + 1], stats=stats[t:t + 1])
        out.append([host(v) for v in (traj, stats, sim.get_state(), sim.get_flags())])
        sim.close()
    for u, w in zip(*out):
        np.testing.assert_array_equal(u, w)
    assert sorted(np.flatnonzero(out[0][3])) == sorted({7, 100, 300, E - 1})
    assert list(out[0][1][:, 3]) == [2, 3, 3, 4]


@pytest.mark.parametrize("fleet,S,mode,T,piece", [
    ("mixed", 16, "rollout", 16, 8), ("plain_mixed", 16, "rollout", 17, 15),
    ("plain_mixed", 2, "step", 6, 3),
])
def test_launch_per_class_equals_one_launch(mgmod, fleet, S, mode, T, piece):
    """A call long enough for a launch per class on a large sim equals the same control steps
    in shorter calls, which take all classes in one launch, bitwise; in rollouts with envs
    that go non-finite part-way.  The call is made twice from the same start (a rollout's
    second one is a replay)."""
    classes, E = FLEETS[fleet], 2048 * 256 + 3
    assert torch.cuda.get_device_properties(0).multi_processor_count <= 256
    cls, x0, _, mult = _inputs(classes, E, 1, 71)
    gen = torch.Generator(device="cuda").manual_seed(72)
    act = torch.rand(T, 8, E, device="cuda", generator=gen) * 2.4 - 1.2
    if mode == "rollout":
        act[0, 0, 7] = act[piece, 1, 100] = act[T - 1, 0, E - 1] = float("nan")
    say("launch per class", fleet, mode)
    sim = mgmod.Sim(classes, E, 0.005, S, env_class=cls)
    fn = sim.rollout if mode == "rollout" else sim.step
    x0, mult = dev(x0), dev(mult)

    def run(n, traj, stats):
        sim.reset(state=x0, param_mult=mult)
        traj.fill_(-1.0)
        for t in range(0, T, n):
            fn(act[t:t + n], traj=traj[t:t + n], stats=stats[t:t + n])
        return [v.clone() for v in (traj, stats, sim.get_state(), sim.get_flags())]

    bufs = (torch.empty(T, x0.shape[0], E, device="cuda"),
            torch.empty(T, 4, dtype=torch.float64, device="cuda"))
    want = run(piece, *bufs)
    for _ in range(2):
        for name, u, w in zip(("traj", "stats", "state", "flags"), run(T, *bufs), want):
            assert torch.equal(u.view(torch.uint8), w.view(torch.uint8)), name
    sim.close()


@pytest.mark.parametrize("fleet,task,m,sizes", [
    ("heavy", "helix", 4, (1, 17, 16384)),
    ("bluerov2", "lemniscate", 1, (33,)),
    ("three", "circle", 16, (49,)),
    ("mixed", "circle", 5, (2, 1001)),
    ("lag_and_not", "station", 3, (1001,)),
])
def test_task_quad_equals_one_env_per_lane(mgmod, fleet, task, m, sizes):
    """Task steps with one env per quad of lanes and per lane: observations, errors, done flags
    and everything a restart writes, bitwise; episodes end by their length, by the error bound
    and by a non-finite state."""
    classes, T = FLEETS[fleet], 5
    cls, x0, act, mult = _inputs(classes, BIG, T, 61)
    act[1, 0, 0] = act[1, 0, 20] = np.nan
    rng = np.random.default_rng(65)
    x1 = random_states(BIG, x0.shape[0], 66)
    center, phase, yaw = (rng.standard_normal(n).astype(np.float32)
                          for n in ((3, BIG), (BIG,), (BIG,)))
    say("task", fleet, task, m)

    def run(E):
        sim = mgmod.Sim(classes, E, 0.005, 3, env_class=cls[:E])
        sim.reset(state=dev(x0[:, :E]), param_mult=dev(mult[:, :E]))
        sim.task_configure(dict(task=task, lookahead=m, radius=1.0, omega=0.5, climb_rate=0.1,
                                episode_steps=4, max_error=2.5),
                           dev(center[:, :E]), dev(phase[:E]), dev(yaw[:E]))
        out = [host(sim.task_observe())]
        for t in range(T):
            kw = dict(reset_state=dev(x1[:, :E]), reset_mult=dev(mult[::-1, :E].copy())) \
                if t % 2 else {}
            out += [host(v) for v in sim.task_step(dev(act[t, :, :E]), **kw)]
        out += [host(sim.get_state()), host(sim.get_params()), host(sim.get_flags()),
                host(sim.task_counters())]
        sim.close()
        return out

    big = run(BIG)
    dones = np.stack(big[3::3][:T])
    assert (dones == 1).any() and (dones == 2).any() and (dones == 0).any()
    for E in sizes:
        say("  envs", E)
        for i, (u, w) in enumerate(zip(run(E), big)):
            np.testing.assert_array_equal(u, w[..., :E], err_msg=str(i))
