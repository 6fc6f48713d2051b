"""The C ABI's host code on the CPU, over a HIP runtime of the test's own
(tests/native/fake_hip.h): what the library launches, copies and allocates, in which order and with
which addresses."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_2407_20026_amd")
OUT = os.path.join(PACKAGE, "_build", "api_checks")


@pytest.fixture(scope="module")
def program():
    from paper_2407_20026_amd import LIB_PATH, build
    if not os.path.exists(LIB_PATH):
        build.build()
    os.makedirs(os.path.dirname(OUT), exist_ok=True)
    cmd = [build.hipcc(), "-x", "hip", "--offload-host-only", "-fPIC", "-O1", "-g", "-std=c++17",
           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PACKAGE, "csrc"), "-c",
           os.path.join(ROOT, "tests", "native", "api_checks.cpp"), "-o", OUT + ".o"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    # the program's own HIP functions come before the runtime's in the order of lookup
    cmd = ["g++", "-rdynamic", "-pthread", OUT + ".o", "-L", PACKAGE, "-lhipsso",
           "-Wl,-rpath," + PACKAGE, "-o", OUT]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return OUT


@pytest.mark.parametrize("check", [
    "ended_before_a_launch", "mixed_recurrences_named_anew", "one_call_ends_a_solve",
    "iterations_are_steps", "a_call_with_several", "allocations_that_fail",
    "launches_that_fail", "ended_on_another_device", "no_host_memory_for_a_plan",
    "memory_left_for_others"])
def test_host_code(program, check):
    r = subprocess.run([program, check], capture_output=True, text=True, timeout=120)
    print(r.stdout[-4000:], r.stderr[-2000:])
    assert r.returncode == 0 and r.stdout.strip().endswith("ok (0 failures)")
