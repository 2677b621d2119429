"""The launchers' choice of kernels and grids in the built library, without a GPU (tests/dispatch_driver.cpp: dry runs)."""
import os
import shutil
import subprocess

import pytest

from paper_2304_11745_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not on PATH")
def test_launchers_choose_what_their_rules_say(tmp_path):
    exe = str(tmp_path / "dispatch_driver")
    cmd = ["hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-x", "hip", os.path.join(HERE, "dispatch_driver.cpp"), "-x", "none", build.LIB, "-Wl,-rpath," + os.path.dirname(build.LIB), "-o", exe]
    built = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert built.returncode == 0, built.stderr[-4000:]
    ran = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert ran.returncode == 0, (ran.stdout + ran.stderr)[-4000:]
    assert "all checks held" in ran.stdout
