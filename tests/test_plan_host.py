"""The plans' host logic of the C ABI on the CPU (tests/host/plan_main.cpp): the
launch chosen for a caller who names none, and what an execution clears after one
that failed, with the HIP runtime and the kernel launchers replaced by
stand-ins."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = "/opt/rocm"
CLANG = os.path.join(ROCM, "llvm", "bin", "clang++")


@pytest.mark.skipif(not os.path.exists(CLANG) or shutil.which("g++") is None,
                    reason="ROCm clang++ not available")
def test_plans(tmp_path):
    from test_sanitizers import CSRC, INC, SAN, _write_bundle   # CPU-only files
    _write_bundle(str(tmp_path / "inputs.bin"))
    inc = ["-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROCM, "include"), "-I" + INC, "-I" + CSRC,
           "-I" + SAN]
    api = str(tmp_path / "api.o")
    subprocess.run([CLANG, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-fPIC", *inc,
                    "-c", os.path.join(CSRC, "sde_api.cpp"), "-o", api], check=True)
    exe = str(tmp_path / "plans")
    subprocess.run(["g++", "-std=c++17", "-O1", *inc, os.path.join(ROOT, "tests", "host", "plan_main.cpp"),
                    os.path.join(CSRC, "sde_tables.cpp"), api, "-o", exe,
                    "-Wl,--unresolved-symbols=ignore-all"], check=True)   # (the device image)
    r = subprocess.run([exe, str(tmp_path / "inputs.bin")], capture_output=True, text=True,
                       timeout=120)
    print(r.stdout, r.stderr)
    assert r.returncode == 0 and "done: 0 failures" in r.stdout
