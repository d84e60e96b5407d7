"""The cache of sweep plans on the host: a plan in use outlives its eviction
(AddressSanitizer build of the planner, look-ups in the order of a step)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2011_02991_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan_cache") / "plan_cache")
    subprocess.run(["g++", "-g", "-O1", "-std=c++17", "-fsanitize=address", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-I" + CSRC, os.path.join(HERE, "plan_cache.cpp"),
                    os.path.join(CSRC, "sweep.cpp"), os.path.join(CSRC, "circuit.cpp"), "-o", exe], check=True)
    return exe


def test_plans_in_use_outlive_their_eviction(program):
    r = subprocess.run([program], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.split()[-1] == "ok", r.stdout + r.stderr
