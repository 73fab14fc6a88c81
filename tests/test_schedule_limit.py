"""The work list under a limit of its cost (host code, no GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_limit(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc) and not shutil.which("hipcc"):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "limit_check")
    subprocess.check_call([hipcc, "--cuda-host-only", "-x", "hip", "-std=c++20", "-O1",
                           "-I", os.path.join(ROOT, "paper_2401_17074_amd", "csrc"),
                           os.path.join(ROOT, "tests", "schedule_limit_check.cpp"), "-o", exe],
                          stderr=subprocess.DEVNULL)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout) > 100
