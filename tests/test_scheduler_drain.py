"""The serving scheduler waits for the executor before it releases the jobs of a
tick that failed: tests/cpu/scheduler_drain_test.cpp, built with g++ under
AddressSanitizer and UndefinedBehaviorSanitizer."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2412_14671_amd", "csrc")


def test_nothing_is_released_in_flight(tmp_path):
    exe = str(tmp_path / "scheduler_drain_test")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=undefined", "-I", CSRC,
                    os.path.join(CSRC, "scheduler.cpp"),
                    os.path.join(ROOT, "tests", "cpu", "scheduler_drain_test.cpp"),
                    "-lpthread", "-o", exe], check=True, capture_output=True, text=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:verify_asan_link_order=0",
               UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120, env=env)
    print(r.stdout, r.stderr[-4000:])
    assert r.returncode == 0
    assert "all passed" in r.stdout
