"""GPU check of the order in which the blocks of interleaved classes run, one env per lane
(ClassSegs::order): fleets of 3 and 16 classes of very different sizes, one of them empty and
one with a single env, against the same envs grouped class by class (no such order), bitwise,
through steps, rollouts, the split scheme and task steps."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.gpu_util import dev, say                                            # noqa: E402
from workloads import (BLUEROV2, BLUEROV2_HEAVY, param_multipliers,            # noqa: E402
                       random_states, vehicle_variant)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_classes,E", [(3, 20011), (16, 70001)])
def test_interleaved_blocks_equal_grouped_ones(n_classes, E):
    from paper_2410_14117_amd import mg
    lag = [vehicle_variant(v, thr_map=1, thr_tau=0.05) for v in (BLUEROV2, BLUEROV2_HEAVY)]
    classes = [dict(lag[k % 2], mass=11.0 + 0.25 * k,
                    added_mass=[0.4 * m for m in lag[k % 2]["added_mass"]])
               for k in range(n_classes)]
    rng = np.random.default_rng(171)
    share = np.r_[0.0, 1.0, np.linspace(1, 6, n_classes - 2)] if n_classes > 3 \
        else np.array([0.15, 0.85, 0.0])
    cls = rng.choice(n_classes, E, p=share / share.sum()).astype(np.int32)
    cls[E // 2] = 0 if n_classes > 3 else 2      # the only env of its class
    group = np.argsort(cls, kind="stable")
    D, S, T = 21, 2, 3
    x0, mult = random_states(E, D, 172), param_multipliers(E, 0.2, 173)
    x0[19:, cls % 2 == 0] = 0
    act = (rng.random((T, 8, E), dtype=np.float32) * 2.4 - 1.2)
    say("interleaved blocks", n_classes, E)
    res = []
    for sel in (np.arange(E), group):
        sim = mg.Sim(classes, E, 0.005, S, env_class=cls[sel])
        xs, ms, a = dev(x0[:, sel]), dev(mult[:, sel]), dev(act[:, :, sel])
        out = []
        for mode in ("step", "rollout", "step_split"):
            sim.reset(state=xs, param_mult=ms)
            traj = torch.full((T, D, E), -1.0, device="cuda")
            stats = torch.zeros((T, 4), dtype=torch.float64, device="cuda")
            getattr(sim, mode)(a, traj=traj, **({} if mode == "step_split" else
                                                {"stats": stats}))
            out += [traj, sim.get_state(), stats]
        sim.task_configure({"task": "helix", "lookahead": 3, "radius": 2.0, "omega": 0.5,
                            "climb_rate": 0.1, "episode_steps": 2},
                           center=dev(x0[:3, sel]), phase=dev(x0[3, sel]))
        for t in range(T):
            out += [v.clone() for v in sim.task_step(a[t], reset_state=xs)]
        out.append(sim.get_state())
        sim.close()
        res.append(out)
    perm = torch.from_numpy(group).cuda()
    for i, (u, w) in enumerate(zip(*res)):
        if u.dtype == torch.float64:             # partials of the same blocks, in the same order
            assert torch.equal(u, w), i
        else:
            assert torch.equal(u.index_select(-1, perm), w), i
