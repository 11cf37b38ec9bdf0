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


@pytest.mark.parametrize("name", ["merge_bins", "split_length", "tuning_candidates",
                                  "line_multipliers", "over_threads"])
def test_plan(check, name):
    p = subprocess.run([check, name], capture_output=True, text=True, timeout=60)
    assert p.returncode == 0, p.stdout + p.stderr


def test_thread_local_storage_holds_messages_only():
    """The first use of a loaded library's thread-local storage in a thread
    allocates it, so the no-allocation call may use none on its way to NRT_OK:
    the one thread-local is the message of a failed call."""
    import paper_2512_12466_amd as nrt
    out = subprocess.run(["readelf", "-sW", nrt.LIB_PATH], check=True, capture_output=True,
                         text=True).stdout
    tls = [line.split()[-1] for line in out.splitlines() if " TLS " in line]
    assert tls and all("g_init_error" in s for s in tls), tls
