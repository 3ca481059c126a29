"""The planner of the 3-D passes (columns cut into pieces), checked on the host
by a compiled driver (tests/host/steps_check.cpp)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_pieces_cover_the_columns_in_the_rounds_counted(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = tmp_path / "steps_check"
    cmd = [cxx, "-O2", "-std=c++17", os.path.join(HERE, "host", "steps_check.cpp"), "-o", str(exe)]
    build = subprocess.run(cmd, capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-2000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout[-2000:]
    assert "bad=0" in run.stdout
