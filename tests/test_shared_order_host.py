"""The order of the shared-sum form's FP32 additions, read from its device tables on the host: no
series carries more rounding than channel by channel in blocks of 32, whatever its bundles are."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1401_8258_amd", "csrc")


def test_no_series_rounds_more_than_channel_by_channel(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = tmp_path / "shared_order"
    r = subprocess.run([gxx, "-std=c++17", "-O2", "-ffp-contract=off", os.path.join(ROOT, "tests", "shared_order_main.cpp"),
                        os.path.join(CSRC, "plan.cpp"), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    assert re.search(r"^ok \d+$", r.stdout, re.M)
