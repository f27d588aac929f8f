"""GPU checks of the kernels with one env per quad of lanes where a fleet, a vehicle or a call
is out of the ordinary: a declared class without envs behind an odd number of groups of 16,
thruster states that are not finite where the velocities are, the statistics of very long
calls, and thruster lags that the split scheme's time step makes unstable."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.gpu_util import dev, host, rel_err, say                             # noqa: E402
from workloads import (BLUEROV2, BLUEROV2_HEAVY, actions, param_multipliers,   # noqa: E402
                       random_states, vehicle_variant)

pytestmark = pytest.mark.gpu

LAG_HEAVY = vehicle_variant(BLUEROV2_HEAVY, thr_map=1, thr_tau=0.05)


@pytest.fixture(scope="module")
def mgmod():
    from paper_2410_14117_amd import mg
    mg.lib()
    return mg


@pytest.mark.parametrize("E", [4585, 5001])
@pytest.mark.parametrize("where", ["first", "last"])
def test_adjoint_of_odd_groups_with_an_empty_class(mgmod, E, where):
    """287 and 313 groups of 16 envs (the paired sweep of 256 compute units, its last block's
    second half without a group) of Heavies, one sub-step, with a lagged class that no env
    belongs to: the gradients, recomputed and from the trajectory, are those of the one-class
    sim, bitwise."""
    T, K = 5, 2
    x0, mult = random_states(E, 13, 81), param_multipliers(E, 0.2, 82)
    act = actions(T, 8, E, 83)
    g = np.random.default_rng(84).standard_normal((T, 13, E)).astype(np.float32)
    pad = lambda a: np.concatenate([a, np.zeros(a.shape[:-2] + (8, E), np.float32)], axis=-2)
    fleets = {"one": ([BLUEROV2_HEAVY], 0, x0, g),
              "two": ([LAG_HEAVY, BLUEROV2_HEAVY] if where == "first"
                      else [BLUEROV2_HEAVY, LAG_HEAVY], int(where == "first"), pad(x0), pad(g))}
    res = {}
    for name, (classes, cls, xs, gs) in fleets.items():
        say("adjoint with an empty class", where, E, name)
        sim = mgmod.Sim(classes, E, 0.01, 1, env_class=np.full(E, cls, np.int32))
        sim.reset(state=dev(xs), param_mult=dev(mult))
        a, traj = dev(act), torch.full((T,) + xs.shape, -1.0, device="cuda")
        ckpt, _ = sim.adj_forward(a, K, traj=traj)
        res[name] = [host(traj)]
        for kw in ({}, {"traj": traj}):
            res[name] += [host(v) for v in sim.adj_backward(ckpt, a, K, dev(gs), **kw)]
        sim.close()
    for i, (u, w) in enumerate(zip(res["two"], res["one"])):
        if u.shape != w.shape:
            assert (u[..., 13:, :] == 0).all(), i
            u = u[..., :13, :]
        np.testing.assert_array_equal(u, w, err_msg=str(i))


@pytest.mark.parametrize("T", [8, 10])
@pytest.mark.parametrize("mode", ["step", "rollout", "steps"])
def test_thruster_states_that_overflow_freeze_their_env(mgmod, mode, T):
    """A thruster without effect (its direction is zero) whose lag is unstable at this time step
    overflows in the eighth control step while the velocities stay finite; an env that is not
    steppable holds a NaN thruster state.  State, flags, counts and trajectory with one env per
    quad of lanes are those with one env per lane, bitwise."""
    heavy = vehicle_variant(BLUEROV2_HEAVY, thr_tau=0.0005)
    heavy["thr_dir"] = list(heavy["thr_dir"][:7]) + [(0.0, 0.0, 0.0)]
    big, E = 20000, 40
    x0, mult = random_states(big, 21, 91), param_multipliers(big, 0.2, 92)
    x0[13:] = 0
    act = np.zeros((T, 8, big), np.float32)
    act[:, 7, 3] = act[:, 7, 18] = 0.5
    mult[4:7, 5], x0[14, 5] = -9.0, np.nan
    res = []
    for n in (E, big):
        say("overflowing thruster states", mode, T, n)
        sim = mgmod.Sim(heavy, n, 0.005, 2)
        sim.reset(state=dev(x0[:, :n]), param_mult=dev(mult[:, :n]))
        a, traj = dev(act[:, :, :n]), torch.full((T, 21, n), -1.0, device="cuda")
        stats = torch.empty((T, 4), dtype=torch.float64, device="cuda")
        if mode == "steps":
            for t in range(T):
                sim.step(a[t:t + 1], traj=traj[t:t + 1], stats=stats[t:t + 1])
        else:
            getattr(sim, mode)(a, traj=traj, stats=stats)
        res.append([host(v) for v in (traj, sim.get_state(), sim.get_flags())] +
                   [host(stats)[:, 3]])
        sim.close()
    small, ref = res
    for name, u, w in zip(("traj", "state", "flags"), small, ref):
        np.testing.assert_array_equal(u, w[..., :E], err_msg=name)
    np.testing.assert_array_equal(small[3], ref[3])
    assert list(np.flatnonzero(ref[2])) == [3, 5, 18] and list(ref[2][[3, 5, 18]]) == [1, 3, 1]
    assert list(ref[3][:8]) == [1] * 7 + [3]


def test_statistics_of_a_long_call_take_bounded_memory(mgmod):
    """4096 control steps of 16 384 envs with statistics in one call: the device memory the sim
    takes for them stays below 64 MiB (as FP64 partials of every 16 envs they would be 128 MiB),
    and the call's results are those of two calls of half the length."""
    E, T = 16384, 4096
    one = dict(BLUEROV2, thr_pos=BLUEROV2["thr_pos"][:1], thr_dir=BLUEROV2["thr_dir"][:1])
    x0 = dev(random_states(E, 13, 101))
    act = torch.zeros((T, 1, E), device="cuda")
    act[::3] = 0.25
    say("statistics of a long call")
    res = []
    for n in (T, T // 2):
        sim = mgmod.Sim(one, E, 0.01, 1)
        sim.reset(state=x0)
        sim.step(act[:1])               # the code is loaded
        sim.reset(state=x0)
        stats = torch.zeros((T, 4), dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        for t in range(0, T, n):
            sim.step(act[t:t + n], stats=stats[t:t + n])
        torch.cuda.synchronize()
        took = free - torch.cuda.mem_get_info()[0]
        print("control steps a call", n, "MiB taken", took / 2**20)
        assert took <= 64 << 20
        res.append((host(sim.get_state()), host(stats)))
        assert not host(sim.get_flags()).any()
        sim.close()
    np.testing.assert_array_equal(res[0][0], res[1][0])
    # FP64 sums of the same values in another order
    np.testing.assert_allclose(res[0][1], res[1][1], rtol=1e-12)


@pytest.mark.parametrize("E", [40, 20000])
def test_split_lag_factor_beyond_fp32(mgmod, oracle, E):
    """Split steps of 41 sub-steps whose lag maps f - f_cmd to -9 (f - f_cmd): over a control
    step that is 1.3e39, more than FP32 holds.  Thrusters at rest under zero throttles stay at
    rest, and 1e-30 N of a thruster without effect becomes -1.3e9 N, as when the lag is stepped.
    Against the oracle within the 1e-4 that 80 sub-steps of the scheme are held to."""
    vs = [vehicle_variant(v, thr_tau=0.0005, added_mass=[0.4 * m for m in v["added_mass"]])
          for v in (BLUEROV2, BLUEROV2_HEAVY)]
    vs[1]["thr_dir"] = list(vs[1]["thr_dir"][:7]) + [(0.0, 0.0, 0.0)]
    cls = (np.arange(E) % 3 == 0).astype(np.int32)
    x0, mult = random_states(E, 21, 111), param_multipliers(E, 0.2, 112)
    x0[13:] = 0
    x0[20, 3] = 1e-30
    act = np.zeros((2, 8, E), np.float32)
    say("split, lag factor beyond FP32", E)
    sim = mgmod.Sim(vs, E, 0.005, 41, env_class=cls)
    sim.reset(state=dev(x0), param_mult=dev(mult))
    traj = torch.full((2, 21, E), -1.0, device="cuda")
    sim.step_split(dev(act), traj=traj)
    got, xT = host(traj), host(sim.get_state())
    sim.close()
    n = min(E, 64)
    ref = oracle.split_rollout(vs, x0[:, :n], act[:, :, :n], 41, 0.005, env_class=cls[:n],
                               mult=mult[:, :n], want_traj=True)["traj"]
    assert rel_err(got[0, :, :n], ref[0]) <= 1e-4
    assert ref[0, 20, 3] < -1e9
    rest = np.arange(n) != 3
    assert rel_err(got[1][:, :n][:, rest], ref[1][:, rest]) <= 1e-4
    np.testing.assert_array_equal(xT, got[1])
