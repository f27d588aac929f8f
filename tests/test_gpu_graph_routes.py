"""GPU checks of the rollouts that are captured into HIP graphs and replayed: the per-sub-step
comparator, and fleets in which some classes have a lag and some have none."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.gpu_util import TOL_ONE_STEP, dev, host, rel_err, say               # noqa: E402
from workloads import (BLUEROV2, BLUEROV2_HEAVY, actions, initial_state,       # noqa: E402
                       vehicle_variant)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mgmod():
    from paper_2410_14117_amd import mg
    mg.lib()
    return mg


def test_plain_rollouts_beyond_the_graph_cache(mgmod):
    """70 per-sub-step rollouts into 70 different trajectory buffers (more than the 64 cached
    graphs), then the first five again, evicted and captured anew: every one writes the same
    trajectory, that of the fused steps."""
    E, T = 64, 2
    x0, act = dev(initial_state(E, 13, 121)), dev(actions(T, 6, E, 122))
    sim = mgmod.Sim(BLUEROV2, E, 0.005, 2)
    say("plain rollouts beyond the graph cache")
    big = torch.zeros((70, T, 13, E), device="cuda")
    for i in list(range(70)) + list(range(5)):
        big[i].zero_()
        sim.reset(state=x0)
        sim.rollout(act, traj=big[i], plain=True)
    want = torch.empty((T, 13, E), device="cuda")
    sim.reset(state=x0)
    sim.step(act, traj=want)
    want = host(want)
    got = host(big)
    for i in range(70):
        assert rel_err(got[i], want) <= TOL_ONE_STEP, i
        np.testing.assert_array_equal(got[i], got[0], err_msg=str(i))
    sim.close()


def test_replays_between_eager_work_and_growing_statistics(mgmod):
    """A part-lagged fleet of 20 000 envs: a rollout captured once and replayed three times with
    eager steps, a reset and a synchronisation between, then a longer rollout whose statistics
    grow the partials' buffer (every graph is dropped), then the first again.  Trajectory,
    statistics and state of each equal those of single steps, bitwise."""
    E, T, S = 20000, 6, 2
    heavy = vehicle_variant(BLUEROV2_HEAVY, thr_map=1, thr_tau=0.05)
    cls = (np.arange(E) % 2).astype(np.int32)
    x0, act = dev(initial_state(E, 21, 131)), dev(actions(T, 8, E, 132))
    sim = mgmod.Sim([BLUEROV2, heavy], E, 0.005, S, env_class=cls)
    traj = torch.empty((T, 21, E), device="cuda")
    stats = torch.empty((T, 4), dtype=torch.float64, device="cuda")
    say("graph replays of a part-lagged fleet")
    sim.reset(state=x0)
    for t in range(T):
        sim.step(act[t:t + 1], traj=traj[t:t + 1], stats=stats[t:t + 1])
    want_traj, want_stats = traj.clone(), stats.clone()
    for i, n in enumerate((2, 2, 2, T, 2, T)):
        say("  call", i, "control steps", n)
        sim.reset(state=x0)
        traj.zero_()
        stats.zero_()
        sim.rollout(act[:n], traj=traj[:n], stats=stats[:n])
        np.testing.assert_array_equal(host(traj[:n]), host(want_traj[:n]))
        np.testing.assert_array_equal(host(stats[:n]), host(want_stats[:n]))
        np.testing.assert_array_equal(host(sim.get_state()), host(want_traj[n - 1]))
        sim.step(act[3:5])
        torch.cuda.synchronize()
    sim.close()
