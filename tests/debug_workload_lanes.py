"""A small pass over the kernel families with one env per lane (sims too large for those with
one env per quad of lanes): the step of all classes in one launch and of one class at a time,
rollouts, Gym tasks, split scheme, the adjoint's forward, recomputation and reverse sweeps, run
with whichever libmg the binding loads (MG_LIBRARY selects libmg_debug.so).  Used by
tests/test_gpu_debug_lanes.py as debug_workload.py is by tests/test_gpu_debug.py.

    python tests/debug_workload_lanes.py OUT.npz     (writes the arrays and the words)
"""
import os
import sys

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


def sizes():
    """Envs of the stepped sims (just beyond one quad wave per SIMD), and of the adjoints (that,
    and just beyond one wave per SIMD with one env per lane, where the sweeps take two)."""
    import torch
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    return n_cu * 64 + 37, (n_cu * 64 + 37, n_cu * 256 + 5)


def run():
    import torch
    from paper_2410_14117_amd import mg
    from workloads import (BLUEROV2, BLUEROV2_HEAVY, vehicle_variant, initial_state, actions,
                           param_multipliers)
    dev = "cuda:0"
    lag = [vehicle_variant(v, thr_map=1, thr_tau=0.05) for v in (BLUEROV2, BLUEROV2_HEAVY)]
    out, words = {}, {}
    E, adj = sizes()
    cls = (np.arange(E) % 3 == 0).astype(np.int32)
    for name, classes in (("alike", lag), ("part", [BLUEROV2, lag[1]])):
        sim = mg.Sim(classes, E, 0.005, 2, env_class=cls)
        D, N = sim.state_dim, sim.action_dim
        x0 = torch.from_numpy(initial_state(E, D, 911)).to(dev)
        mult = torch.from_numpy(param_multipliers(E, 0.2, 912)).to(dev)
        act = torch.from_numpy(actions(5, N, E, 913)).to(dev)
        sim.reset(state=x0, param_mult=mult)
        traj = torch.empty((3, D, E), device=dev)
        stats = torch.empty((3, 4), dtype=torch.float64, device=dev)
        for mode in ("step", "rollout"):
            getattr(sim, mode)(act[:3], traj=traj, stats=stats)
            out[f"{name}_{mode}_traj"] = traj.cpu().numpy()
            out[f"{name}_{mode}_stats"] = stats.cpu().numpy()
        sim.step(act[3:4], plain=True)
        sim.reset(env_ids=torch.arange(0, E, 7, device=dev), state=x0[:, ::7].contiguous())
        out[f"{name}_state"] = sim.get_state().cpu().numpy()
        sim.task_configure({"task": "circle", "lookahead": 4, "radius": 2.0, "omega": 0.5,
                            "episode_steps": 2},
                           center=torch.zeros(3, E, device=dev),
                           phase=torch.linspace(0, 6.0, E, device=dev))
        for k in range(3):
            obs, err, done = sim.task_step(act[k], reset_state=x0)
            for key, v in (("obs", obs), ("err", err), ("done", done)):
                out[f"{name}_task_{key}{k}"] = v.cpu().numpy()
        sim.reset(state=x0, param_mult=mult)
        sim.step_split(act[:2])
        out[f"{name}_split"] = sim.get_state().cpu().numpy()
        words[name] = sim.debug_word()
        sim.close()

    for i, Ea in enumerate(adj):
        T = 4
        sa = mg.Sim(BLUEROV2, Ea, 0.01, 1)
        xa = torch.from_numpy(initial_state(Ea, 13, 914)).to(dev)
        aa = torch.from_numpy(actions(T, 6, Ea, 915)).to(dev)
        g = torch.from_numpy(np.random.default_rng(916).standard_normal((T, 13, Ea))
                             .astype(np.float32)).to(dev)
        for form, K, with_traj in (("traj", 2, True), ("whole", 2, False), ("segment", 4, False)):
            sa.reset(state=xa)
            tra = torch.empty((T, 13, Ea), device=dev)
            ck, _ = sa.adj_forward(aa, K, traj=tra)
            res = sa.adj_backward(ck, aa, K, g, **({"traj": tra} if with_traj else {}))
            for key, v in zip(("traj", "act", "theta", "x0"), (tra,) + tuple(res)):
                out[f"adj{i}_{form}_{key}"] = v.cpu().numpy()
        words[f"adj{i}"] = sa.debug_word()
        sa.close()
    torch.cuda.synchronize()
    return out, words


if __name__ == "__main__":
    res, w = run()
    np.savez(sys.argv[1], **res, **{f"word_{k}": np.uint32(v) for k, v in w.items()})
    print("debug workload done:", {k: int(v) for k, v in w.items()}, flush=True)
