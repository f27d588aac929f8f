"""GPU checks of whole-sim resets, parameters, states and read-backs of fleets whose classes are
interleaved env by env, at sizes and class counts on either side of the rules that choose the
order in which the kernels go through the envs (runtime.hip: reset_internal; kernels_step.hip:
launch_scatter_in)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.gpu_util import dev, say                                            # noqa: E402
from workloads import (BLUEROV2, BLUEROV2_HEAVY, param_multipliers,            # noqa: E402
                       random_states, vehicle_variant)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_classes,E", [(3, 1001), (3, 200003), (3, 600011), (8, 1001), (8, 300007),
                                         (8, 200003)])
def test_whole_resets_equal_resets_by_id(n_classes, E):
    """Parameters, states and flags after a reset of every env, and after set_params and
    set_state, are bitwise those of the same inputs reset by env ids, one column each."""
    from paper_2410_14117_amd import mg
    lag = [vehicle_variant(v, thr_map=1, thr_tau=0.05) for v in (BLUEROV2, BLUEROV2_HEAVY)]
    classes = [dict(lag[k % 2], mass=11.0 + 0.25 * k) for k in range(n_classes)]
    cls = np.random.default_rng(161).integers(0, n_classes, E).astype(np.int32)
    x0, mult = random_states(E, 21, 162), param_multipliers(E, 0.2, 163)
    mult[4:7, 77] = -9.0             # mass matrix not positive definite
    x0, mult, ids = dev(x0), dev(mult), torch.arange(E, device="cuda")
    say("interleaved resets", n_classes, E)
    sims = [mg.Sim(classes, E, 0.005, 2, env_class=cls) for _ in range(2)]
    sims[0].reset(state=x0, param_mult=mult)
    sims[1].reset(env_ids=ids, state=x0, param_mult=mult)

    def same(what):
        for name in ("get_state", "get_params", "get_flags"):
            u, w = (getattr(s, name)() for s in sims)
            assert torch.equal(u, w), (what, name)
        assert sims[0].get_flags().nonzero().flatten().tolist() == [77]

    same("reset")
    act = torch.full((2, 8, E), 0.3, device="cuda")
    for s in sims:
        s.step(act)
    same("step")
    sims[0].reset(param_mult=mult)
    sims[1].reset(env_ids=ids, param_mult=mult)
    same("reset of the parameters")
    params = sims[1].get_params() * 1.0
    sims[0].reset()
    sims[0].set_params(params)
    sims[1].set_params(params)
    for s in sims:
        s.set_state(x0)
    same("set_params, set_state")
    lagged = torch.tensor([19, 21], device="cuda")[torch.from_numpy(cls % 2).cuda().long()]
    rows = torch.arange(21, device="cuda")[:, None] < lagged[None]
    assert torch.equal(torch.where(rows, sims[0].get_state(), 0.0), torch.where(rows, x0, 0.0))
    for s in sims:
        s.close()
