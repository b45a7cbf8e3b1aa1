"""Estimated marching times of served requests (csrc/serve.cpp), no GPU:
tests/native/serve_estimate.cpp on the fake executor of the scheduler's test."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRCS = [os.path.join(ROOT, "tests", "native", f) for f in ("fake_device.cpp", "serve_estimate.cpp")]
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_estimates_follow_the_request(tmp_path):
    exe = str(tmp_path / "serve_estimate")
    res = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROCM, "include")]
                         + SRCS + ["-o", exe, "-lpthread"], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    res = subprocess.run([exe], capture_output=True, text=True, timeout=240)
    assert res.returncode == 0 and "serve_estimate: ok" in res.stdout, res.stdout + res.stderr
