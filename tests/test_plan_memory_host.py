"""Plan creation where host memory is short (tests/plan_memory_main.cpp): no C++ exception leaves it."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_a_table_that_does_not_fit_memory_is_no_abort(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = tmp_path / "plan_memory"
    r = subprocess.run([gxx, "-std=c++17", "-O2", "-ffp-contract=off", os.path.join(ROOT, "tests", "plan_memory_main.cpp"),
                        os.path.join(ROOT, "paper_1401_8258_amd", "csrc", "plan.cpp"), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert (r.returncode, r.stdout.strip()) == (0, "ok"), (r.returncode, r.stdout + r.stderr)
