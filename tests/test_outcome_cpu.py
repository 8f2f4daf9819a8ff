"""Waits inside a launch end, whatever becomes of what is waited for, and its waves agree on it (tests/host/outcome.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2006_02924_amd", "csrc")


def test_every_wait_for_an_outcome_ends(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    exe = tmp_path / "outcome"
    subprocess.run([gxx, "-std=c++17", "-O2", "-Wall", "-I", CSRC, os.path.join(ROOT, "tests", "host", "outcome.cpp"), "-o", str(exe),
                    "-lpthread"], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-2000:]
    assert "outcomes ok" in res.stdout
