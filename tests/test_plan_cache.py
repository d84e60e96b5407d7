"""The cache of sweep plans on the host (AddressSanitizer build of the planner,
look-ups in the order of a step): a plan in use outlives its eviction, 128
circuits keep their plans, and one more evicts those not used for the longest time; and the forward
pass of every register has a plan."""
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


@pytest.mark.parametrize("check", ["use", "round", "oldest", "registers"])
def test_plan_cache(program, check):
    r = subprocess.run([program, check], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.split()[-1] == "ok", r.stdout + r.stderr
