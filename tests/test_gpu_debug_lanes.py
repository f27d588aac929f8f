"""The bounds-checked debug build on sims above the range of the kernels with one env per quad
of lanes: tests/debug_workload_lanes.py in the test's process with the release library and in a
child process with the debug library.  Results equal, bitwise, and no check fires; with a
shrunk bound of caller columns (MG_DEBUG_SHRINK) the column check fires in every sim, and the
other envs' results still equal the release build's."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

from tests.gpu_util import say

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, os.path.join(ROOT, "tests"))


@pytest.fixture(scope="module")
def release():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import debug_workload_lanes
    from paper_2410_14117_amd import mg
    if mg.lib().mg_debug_build() != 0:
        pytest.fail("the test process must load the release library")
    say("debug build, one env per lane: release pass")
    return debug_workload_lanes.run()


@pytest.mark.parametrize("shrink", [0, 100])
def test_lane_kernels_of_the_debug_build(release, tmp_path, shrink):
    from paper_2410_14117_amd import mg
    if not os.path.exists(mg.DEBUG_LIB_PATH):
        pytest.fail(f"{mg.DEBUG_LIB_PATH} is missing: python -m paper_2410_14117_amd.build --debug")
    rel, words = release
    assert not any(words.values())
    out = str(tmp_path / "debug.npz")
    env = dict(os.environ, MG_LIBRARY=mg.DEBUG_LIB_PATH)
    if shrink:
        env["MG_DEBUG_SHRINK"] = str(shrink)
    say("debug build, one env per lane: child process, shrink", shrink)
    r = subprocess.run([sys.executable, "-u",
                        os.path.join(ROOT, "tests", "debug_workload_lanes.py"), out],
                       env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    dbg = dict(np.load(out))
    for name in words:
        fired = int(dbg[f"word_{name}"])
        assert (fired & mg.MG_DBG_COLUMN) if shrink else fired == 0, (name, fired)
    for k, v in rel.items():
        if k.endswith("stats"):
            if not shrink:
                assert np.array_equal(dbg[k], v), k
            continue
        n = v.shape[-1] - shrink
        assert np.array_equal(dbg[k][..., :n], v[..., :n], equal_nan=True), k
        if shrink and k.endswith(("_state", "_split")):   # never reset: the zeros of mg_create
            assert (dbg[k][..., n:] == 0).all(), k
