"""The host's launch rules (csrc/launch_plan.h, csrc/brmppi_internal.h), built for the CPU and checked
over all the sizes that they accept (tests/host/launch_plan_test.cpp lists the
checks), under AddressSanitizer + UndefinedBehaviorSanitizer."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "host", "launch_plan_test.cpp")
INC = [os.path.join(ROOT, "include"), os.path.join(ROOT, "paper_2508_05773_amd", "csrc"), "/opt/rocm/include"]


def test_launch_plan(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "launch_plan")
    cmd = [gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-D__HIP_PLATFORM_AMD__",
           *sum((["-I", d] for d in INC), []), SRC, "-o", exe]
    subprocess.run(cmd, check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=240)
    print(r.stdout)
    assert r.returncode == 0, r.stderr[-4000:]
    assert "launch plan: all checks passed" in r.stdout
