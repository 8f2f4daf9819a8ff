"""A call whose second launch fails between the two of the resident pass: the next call of the plan does not take the words that
it left for its own (tests/host/interrupted_pass.cpp: the library's host side with stand-ins for the launches)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2006_02924_amd", "csrc")
HIP = "/opt/rocm/include"


def test_next_call_after_a_failed_second_launch(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir(os.path.join(HIP, "hip")):
        pytest.skip("no g++ or no HIP headers")
    exe = tmp_path / "interrupted_pass"
    # (launches and runtime calls that these calls do not make stay unresolved)
    cmd = [gxx, "-std=c++17", "-O1", "-g", "-Wall", "-D__HIP_PLATFORM_AMD__", "-no-pie", "-Wl,--unresolved-symbols=ignore-all",
           "-I", HIP, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           os.path.join(ROOT, "tests", "host", "interrupted_pass.cpp"), os.path.join(CSRC, "adasum_api.cpp"),
           os.path.join(CSRC, "adasum_plan.cpp"), "-o", str(exe), "-lpthread"]
    subprocess.run(cmd, check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-2000:]
    assert "interrupted passes ok" in res.stdout
