"""The rules that choose a convolution's kernel and its split, built and checked
on the CPU (tests/host/conv_plan_main.cpp)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_03115_amd", "csrc")
ROCM = "/opt/rocm"


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_conv_plans(tmp_path):
    exe = str(tmp_path / "conv_plan")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__",
                    "-I" + os.path.join(ROCM, "include"), "-I" + CSRC,
                    os.path.join(ROOT, "tests", "host", "conv_plan_main.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    assert r.returncode == 0 and "done: 0 failures" in r.stdout
