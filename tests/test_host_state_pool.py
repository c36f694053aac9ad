"""The pool of pinned job states gives up and takes in states without allocating host memory: a
job's destructor hands its state back, and an exception there would end the process."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = """
#include <utility>
#include "runtime.h"
using muster::Ctx;
static_assert(noexcept(std::declval<Ctx&>().give_host_state(nullptr)), "called by ~Job");
static_assert(noexcept(std::declval<Ctx&>().free_host_states()), "called when a context goes");
"""


def test_giving_a_state_back_cannot_throw(tmp_path):
    src = tmp_path / "pool.cpp"
    src.write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-fsyntax-only", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-I",
                    os.path.join(ROOT, "paper_2412_14671_amd", "csrc"), str(src)], check=True)
