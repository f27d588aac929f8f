"""CPU run of the index arithmetic of the kernels with one env per quad of lanes
(fossen_quad.h: quad_env, host and device code): tests/quad_env_check.hip walks the blocks of
fleets with empty classes, the paired reverse sweep's surplus block among them, and requires
every lane's column to exist.  Built for the host with AddressSanitizer and
UndefinedBehaviorSanitizer (GPU code is not instrumented)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_lane_of_a_quad_launch_has_a_column(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "quad_env_check")
    subprocess.check_call([hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950",
                           "-Xarch_host", "-fsanitize=address,undefined",
                           "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2410_14117_amd", "csrc"),
                           os.path.join(ROOT, "tests", "quad_env_check.hip"), "-o", exe],
                          stderr=subprocess.DEVNULL)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(r.stdout, r.stderr[-3000:])
    assert r.returncode == 0 and "0 failures" in r.stdout, r.stdout[-2000:] + r.stderr[-2000:]
