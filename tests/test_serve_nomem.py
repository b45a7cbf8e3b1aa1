"""Allocation failures of the scheduler's tables (csrc/serve.cpp), no GPU:
tests/native/serve_nomem.cpp on the fake executor of the scheduler's test."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRCS = [os.path.join(ROOT, "tests", "native", f) for f in ("fake_device.cpp", "serve_nomem.cpp")]
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
WRAP = ["-Wl,--wrap=" + f for f in ("hipMalloc", "hipFree", "hipHostMalloc", "hipHostFree")]


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_failed_tables_leave_nothing_behind(tmp_path):
    exe = str(tmp_path / "serve_nomem")
    res = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROCM, "include")]
                         + SRCS + WRAP + ["-o", exe, "-lpthread"], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    res = subprocess.run([exe], capture_output=True, text=True, timeout=240)
    assert res.returncode == 0 and "serve_nomem: ok" in res.stdout, (res.returncode, res.stdout + res.stderr)
