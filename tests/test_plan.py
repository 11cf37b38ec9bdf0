"""On the CPU: the plans of csrc/plan.h over the sizes and parameters that the
entry points accept, the ends of their ranges included, where a device run
would not fit or not end."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-Wall", "-Werror",
                    "-I" + os.path.join(ROOT, "paper_2512_12466_amd", "csrc"),
                    "-I" + os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "plan_check.cpp"), "-o", exe, "-lpthread"],
                   check=True)
    return exe


@pytest.mark.parametrize("name", ["merge_bins", "split_length", "tuning_candidates"])
def test_plan(check, name):
    p = subprocess.run([check, name], capture_output=True, text=True, timeout=60)
    assert p.returncode == 0, p.stdout + p.stderr
