"""dg_step's CFL rate slots after a failed launch, on the CPU: host_rate_slots.cpp linked with the
library's host object."""
import os
import subprocess

import pytest

from paper_1602_09079_amd import build as pb

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_time_step_after_a_failed_launch(tmp_path):
    host_o = os.path.join(pb.HERE, "_build", "dg_host.cpp.o")
    if not os.path.exists(host_o):
        pytest.skip("no build objects")
    exe = str(tmp_path / "host_rate_slots")
    # the calls this program does not reach stay unresolved
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-no-pie", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                           "-I", os.path.join(ROOT, "include"), "-I", pb.CSRC,
                           os.path.join(ROOT, "tests", "host_rate_slots.cpp"), host_o, "-o", exe,
                           "-Wl,--unresolved-symbols=ignore-all"])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
