"""The launches of a chunk plan against its chunks one by one (host code)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def test_launches_follow_the_plan(tmp_path):
    cxx = os.environ.get("CXX") or shutil.which("g++")
    if not cxx or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime_api.h")):
        pytest.skip("needs g++ and the HIP runtime API headers")
    exe = str(tmp_path / "merge_plan_check")
    r = subprocess.run([cxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=all", "-D__HIP_PLATFORM_AMD__",
                        f"-I{os.path.join(ROCM, 'include')}",
                        os.path.join(ROOT, "paper_2609_32197_amd", "csrc", "host_plan.cpp"),
                        os.path.join(ROOT, "tests", "hostcheck", "merge_plan_check.cpp"),
                        "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and " 0 failures" in r.stdout, (r.stdout + r.stderr)[-4000:]
