"""Errors that a wait for a stream reports reach the caller: the host runtime over a fake device
on the CPU, built with g++ under AddressSanitizer and UndefinedBehaviorSanitizer:
tests/cpu/level_errors_test.cpp."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2412_14671_amd", "csrc")

pytestmark = pytest.mark.slow


def test_no_error_of_a_wait_is_lost(tmp_path):
    obj = os.path.join(ROOT, "_build", "kernels.o")
    subprocess.run(["make", "-C", CSRC, "../../_build/kernels.o"], check=True, capture_output=True)
    exe = str(tmp_path / "level_errors_test")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Wno-unused-function",
                    "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
                    "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC,
                    os.path.join(ROOT, "tests", "cpu", "level_errors_test.cpp"),
                    os.path.join(CSRC, "runtime.cpp"), os.path.join(CSRC, "scheduler.cpp"), obj,
                    "-L/opt/rocm/lib", "-Wl,-rpath,/opt/rocm/lib", "-lrocprofiler-sdk-roctx",
                    "-lpthread", "-o", exe], check=True, capture_output=True, text=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:verify_asan_link_order=0",
               UBSAN_OPTIONS="print_stacktrace=1")
    env.pop("MUSTER_TUNE_CACHE", None)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300, env=env)
    print(r.stdout, r.stderr[-4000:])
    assert r.returncode == 0
    assert "all passed" in r.stdout
