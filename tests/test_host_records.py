"""The slots that the rotate-back's corner records lead to, planned on the
host (CPU only)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_corner_records_lead_to_nodes_only(tmp_path):
    exe = str(tmp_path / "records")
    csrc = os.path.join(ROOT, "paper_2205_15000_amd", "csrc")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-I", csrc, os.path.join(ROOT, "tests", "asan", "records_harness.cpp"),
                        os.path.join(csrc, "plan.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "OK" in r.stdout, r.stdout
