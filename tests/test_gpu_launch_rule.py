"""GPU checks of calls on either side of the rule that chooses between one launch for all
classes and a launch per class (runtime.hip: one_launch)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.gpu_util import dev, say                                            # noqa: E402
from workloads import (BLUEROV2, BLUEROV2_HEAVY, param_multipliers,            # noqa: E402
                       random_states, vehicle_variant)

pytestmark = pytest.mark.gpu

LAG = [vehicle_variant(v, thr_map=1, thr_tau=0.05) for v in (BLUEROV2, BLUEROV2_HEAVY)]
LIN = [BLUEROV2, BLUEROV2_HEAVY]


@pytest.mark.parametrize("classes,share,E,S,mode,T,piece,with_traj", [
    (LAG, 0.5, 524291, 16, "rollout", 18, 9, True),     # 8 blocks to a CU: beyond 16 steps
    (LAG, 0.5, 140001, 16, "rollout", 6, 3, True),      # 2-8 blocks: from 6 steps on, 3 without
    (LIN, 0.5, 140001, 16, "rollout", 4, 2, True),
    (LAG, 0.02, 131072, 16, "rollout", 6, 3, False),    # the small class in a third round
    (LIN, 0.02, 524291, 16, "rollout", 18, 9, False),   # one class has nearly all
    (LAG, 0.5, 524291, 2, "step", 10, 5, False),        # 2^22 env control steps
    (LIN, 0.5, 524291, 4, "step", 6, 3, False),         # 2^21
    (LIN, 0.5, 524291, 16, "step", 3, 1, True),         # 2^20, trajectory of interleaved classes
    (LIN, 0.02, 140001, 16, "step", 6, 3, True),        # 2^19
])
def test_a_call_equals_its_pieces(classes, share, E, S, mode, T, piece, with_traj):
    """One call on the far side of the rule and the same control steps in shorter calls on the
    near side: trajectory, statistics, state and flags, bitwise; in rollouts with envs that go
    non-finite part-way.  The long call is made twice."""
    from paper_2410_14117_amd import mg
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256
    cls = (np.random.default_rng(141).random(E) < share).astype(np.int32)
    D = 21 if classes is LAG else 13
    x0 = random_states(E, D, 142)
    if classes is LAG:
        x0[19:, cls == 0] = 0
    gen = torch.Generator(device="cuda").manual_seed(143)
    act = torch.rand(T, 8, E, device="cuda", generator=gen) * 2.4 - 1.2
    if mode == "rollout":
        act[0, 0, 7] = act[piece, 1, 100] = act[T - 1, 0, E - 1] = float("nan")
    say("launch rule", E, S, mode, T, piece)
    sim = mg.Sim(classes, E, 0.005, S, env_class=cls)
    x0, mult = dev(x0), dev(param_multipliers(E, 0.2, 144))
    traj = torch.empty((T, D, E), device="cuda") if with_traj else None
    stats = torch.empty((T, 4), dtype=torch.float64, device="cuda")

    def run(n):
        sim.reset(state=x0, param_mult=mult)
        stats.fill_(-1.0)
        if with_traj:
            traj.fill_(-1.0)
        for t in range(0, T, n):
            kw = {"traj": traj[t:t + n]} if with_traj else {}
            getattr(sim, mode)(act[t:t + n], stats=stats[t:t + n], **kw)
        out = [stats, sim.get_state(), sim.get_flags()] + ([traj] if with_traj else [])
        return [v.clone() for v in out]

    want = run(piece)
    for _ in range(2):
        for name, u, w in zip(("stats", "state", "flags", "traj"), run(T), want):
            assert torch.equal(u.view(torch.uint8), w.view(torch.uint8)), name
    sim.close()


def test_a_rollout_of_launches_per_class_is_captured():
    """A rollout of a launch per class and control step, captured (fork, launches, join) and
    replayed three times with eager work and a synchronisation between: bitwise the eager
    rollout."""
    from paper_2410_14117_amd import mg
    E, S, T = 140001, 16, 6
    cls = (np.arange(E) % 2).astype(np.int32)
    x0 = random_states(E, 21, 151)
    x0[19:, cls == 0] = 0
    x0 = dev(x0)
    gen = torch.Generator(device="cuda").manual_seed(152)
    act = torch.rand(T, 8, E, device="cuda", generator=gen) * 2 - 1
    traj = torch.empty((T, 21, E), device="cuda")
    stats = torch.empty((T, 4), dtype=torch.float64, device="cuda")
    sim = mg.Sim(LAG, E, 0.005, S, env_class=cls)
    say("captured rollout")
    sim.reset(state=x0)
    sim.rollout(act, traj=traj, stats=stats)
    want = [v.clone() for v in (traj, stats, sim.get_state())]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sim.rollout(act, traj=traj, stats=stats)
    for i in range(3):
        sim.reset(state=x0)
        traj.zero_()
        stats.zero_()
        graph.replay()
        for u, w in zip((traj, stats, sim.get_state()), want):
            assert torch.equal(u.view(torch.uint8), w.view(torch.uint8)), i
        sim.step(act[:2])
        torch.cuda.synchronize()
    sim.close()
