"""The kernels' bit-level expressions and EDM's root, compiled for the host from
the sources the kernels include (tests/host/bits_check.cpp)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_bits_and_root(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = tmp_path / "bits_check"
    cmd = [cxx, "-O2", "-std=c++17", "-ffp-contract=off", os.path.join(HERE, "host", "bits_check.cpp"), "-o", str(exe)]
    build = subprocess.run(cmd, capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-2000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout[-2000:]
    assert "bad=0" in run.stdout
