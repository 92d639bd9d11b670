"""The backward's passes over the views: a tap offset is used with the map it was
projected for, and each view is gathered and then used once, in order, for every
view count and both lane counts per pixel (CPU)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_offsets_stay_with_their_map(tmp_path):
    exe = str(tmp_path / "check")
    r = subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I",
                        os.path.join(ROOT, "paper_2411_16680_amd", "csrc"),
                        os.path.join(ROOT, "tests", "view_order_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout[-3000:]
