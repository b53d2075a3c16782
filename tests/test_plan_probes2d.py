"""Host logic: the probe lists of the 2D workgroup tiles.  Builds
tests/plan_check_probes2d.cpp with the library's plan source (host code only)
and runs it on random grids."""
import os
import subprocess

import pytest

from test_plan3d import CSRC, HERE, HIPCC, ROOT


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_wg2d_probe_lists(tmp_path):
    exe = str(tmp_path / "plan_check_probes2d")
    cmd = [HIPCC, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I",
           os.path.join(ROOT, "include"), os.path.join(HERE, "plan_check_probes2d.cpp"),
           os.path.join(CSRC, "plan2d.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "0 bad of" in r.stdout, r.stdout[-2000:]
