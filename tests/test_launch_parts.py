"""How many heads a launch takes, on the CPU: the host's split of a batch into launches, built alone and run."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"), reason="no hipcc")
def test_no_launch_outgrows_a_grid_dimension(tmp_path):
    exe = str(tmp_path / "parts")
    cmd = [shutil.which("hipcc") or "/opt/rocm/bin/hipcc", "--cuda-host-only", "-O1", "-std=c++17", "-x", "hip",
           os.path.join(ROOT, "tests", "sanitize", "parts_driver.cpp"), "-o", exe]
    build = subprocess.run(cmd, capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-3000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and "0 mismatches" in run.stdout, run.stdout + run.stderr
