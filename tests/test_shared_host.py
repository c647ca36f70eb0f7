"""The shared-sum form on the host: its device tables (every trial's sample of every channel,
LDS and input bounds, the double buffer) walked under AddressSanitizer and UBSan, and the device
code of its kernels: no scratch, no spills, no packed FP32."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1401_8258_amd", "csrc")


def test_tables_give_every_trial_its_delays(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = tmp_path / "shared_table"
    cmd = [gxx, "-std=c++17", "-O1", "-g", "-ffp-contract=off", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=undefined", os.path.join(ROOT, "tests", "shared_table_main.cpp"),
           os.path.join(CSRC, "plan.cpp"), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:halt_on_error=1")
    env.pop("LD_PRELOAD", None)
    r = subprocess.run([str(exe)], capture_output=True, text=True, env=env, timeout=600)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    assert re.search(r"^ok \d+$", r.stdout, re.M)


def test_device_code_has_no_scratch_spills_or_packed_fp32(tmp_path):
    hipcc = "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("ROCm toolchain not found")
    from paper_1401_8258_amd import build
    asm = tmp_path / "shared.s"
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([hipcc] + flags + ["--cuda-device-only", "-S", "-o", str(asm), os.path.join(CSRC, "shared.hip")],
                   check=True, capture_output=True)
    text = asm.read_text()
    assert len(re.findall(r"\.name:\s+\S*dedisp_shared", text)) == 3
    for key in ("private_segment_fixed_size", "vgpr_spill_count", "sgpr_spill_count"):
        values = re.findall(r"\.%s:\s+(\d+)" % key, text)
        assert values and all(int(v) == 0 for v in values), (key, values)
    assert not re.search(r"\bv_pk_(add|mul|fma)_f32\b", text)
    assert "flat_load" not in text  # a flat load would be waited on with the LDS reads
