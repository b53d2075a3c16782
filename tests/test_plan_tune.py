"""Host logic: the autotuner's trial lengths and the fewest steps of a pass.
Builds
tests/plan_check_tune.cpp with the library's plan source (host code only) and
runs it."""
import os
import subprocess

import pytest

from test_plan3d import CSRC, HERE, HIPCC, ROOT


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_trials_and_passes(tmp_path):
    exe = str(tmp_path / "plan_check_tune")
    cmd = [HIPCC, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I",
           os.path.join(ROOT, "include"), os.path.join(HERE, "plan_check_tune.cpp"),
           os.path.join(CSRC, "plan2d.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "0 bad of" in r.stdout, r.stdout[-2000:]
