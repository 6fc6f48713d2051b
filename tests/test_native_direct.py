"""The direct solver's plan (nested dissection, fronts, work lists) on the CPU, under
AddressSanitizer and UndefinedBehaviorSanitizer: tests/native/direct_checks.cpp checks its
invariants on graphs of every kind and eliminates with it in plain loops."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2407_20026_amd", "csrc")
OUT = os.path.join(ROOT, "paper_2407_20026_amd", "_build", "direct_checks")


def test_plan_invariants_and_elimination():
    os.makedirs(os.path.dirname(OUT), exist_ok=True)
    cmd = ["g++", "-O1", "-g", "-std=c++17", "-pthread", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=all", "-D_GLIBCXX_ASSERTIONS", "-I", CSRC,
           os.path.join(ROOT, "tests", "native", "direct_checks.cpp"),
           os.path.join(CSRC, "direct_plan.cpp"), "-o", OUT]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([OUT], capture_output=True, text=True, timeout=300)
    print(r.stdout[-2000:], r.stderr[-4000:])
    assert r.returncode == 0 and r.stdout.strip().endswith("ok (0 failures)")
