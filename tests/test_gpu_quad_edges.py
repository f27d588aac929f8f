"""GPU checks of the kernels with one env per quad of lanes where a fleet, a vehicle or a call
is out of the ordinary: a declared class without envs behind an odd number of groups of 16."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.gpu_util import dev, host, say                                      # noqa: E402
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
