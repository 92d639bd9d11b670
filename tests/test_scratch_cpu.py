"""The context's workspaces at their limits (CPU, the C-ABI linked with a
stand-in for the HIP runtime): the backward's optional scratch is refused once
and not asked for again, never under capture, is given back to a call that has
to have the room, and does not change the weight gradients' workgroups."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2411_16680_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_workspaces_at_their_limits(tmp_path):
    exe = str(tmp_path / "check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                        os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(CSRC, "capi.cpp"),
                        os.path.join(ROOT, "tests", "scratch_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout[-3000:]
