"""CPU check of the machine code of the adjoint's recomputing sweeps with two waves per SIMD
(built here for gfx950, 6 and 8 thrusters): they have 256 registers and spill for the rest of a
sub-step VJP, which is what their speed hangs on.  The limits are what they spilled before the
VJP was written on 3-vectors; beyond them the sweeps were up to 8 % slower."""
import os
import re
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

# (thrusters, lag, whole rollout recomputed first): registers spilled at most
LIMITS = {(6, 0, 0): 24, (6, 0, 1): 12, (6, 1, 0): 37, (6, 1, 1): 28,
          (8, 0, 0): 26, (8, 0, 1): 20, (8, 1, 0): 37, (8, 1, 1): 30}


@pytest.fixture(scope="module")
def spills(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    from paper_2410_14117_amd import build
    d = tmp_path_factory.mktemp("asm")
    src, out = str(d / "kernels_adjoint.hip"), str(d / "kernels_adjoint.s")
    text = open(os.path.join(build.CSRC, "kernels_adjoint.hip")).read()
    every = " ".join(f"MG_CASE({n})" for n in range(1, 9))
    assert every in text
    with open(src, "w") as f:
        f.write(text.replace(every, "MG_CASE(6) MG_CASE(8)"))
    subprocess.check_call([hipcc, "-S", "--cuda-device-only", *build.CFLAGS, src, "-o", out],
                          stderr=subprocess.DEVNULL)
    meta = open(out).read()
    meta = meta[meta.index("amdhsa.kernels:"):]
    return {re.search(r"\.name:\s+(\S+)", e).group(1):
            int(re.search(r"\.vgpr_spill_count:\s+(\d+)", e).group(1))
            for e in meta.split("\n  - ")[1:] if ".vgpr_spill_count" in e}


@pytest.mark.parametrize("key", sorted(LIMITS))
def test_spills_of_the_two_wave_recomputing_sweeps(spills, key):
    n, lag, whole = key
    name = [k for k in spills if f"k_adj_bwdILi{n}ELb{lag}ELi2ELb{whole}ELb0E" in k]
    assert len(name) == 1
    assert spills[name[0]] <= LIMITS[key], (key, spills[name[0]])
