"""Host transfers of one owner from several threads (csrc/pf_host_copy.h) under
sanitizers, no GPU: the pinned stage is shared, so transfers have to take turns.

tests/native/host_copy_threads.cpp on the fake executor of the scheduler's test
(tests/native/fake_device.cpp): two readers and a writer with fields of
different sizes.  g++ with AddressSanitizer + UndefinedBehaviorSanitizer and
ROCm's clang++ with ThreadSanitizer.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRCS = [os.path.join(ROOT, "tests", "native", f) for f in ("fake_device.cpp", "host_copy_threads.cpp")]
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
FLAGS = ["-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", "-D__HIP_PLATFORM_AMD__",
         "-I" + os.path.join(ROCM, "include")]
CLANG = os.path.join(ROCM, "llvm", "bin", "clang++")


@pytest.mark.parametrize("cxx,san", [("g++", "address,undefined"), (CLANG, "thread")], ids=["asan", "tsan"])
def test_transfers_of_several_threads_take_turns(tmp_path, cxx, san):
    if shutil.which(cxx) is None:
        pytest.skip("needs " + cxx)
    exe = str(tmp_path / "host_copy")
    res = subprocess.run([cxx] + FLAGS + ["-fsanitize=" + san] + SRCS + ["-o", exe, "-lpthread"],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    res = subprocess.run([exe], capture_output=True, text=True, timeout=240)
    assert res.returncode == 0 and "host_copy_threads: ok" in res.stdout, (res.stdout + res.stderr)[-6000:]
