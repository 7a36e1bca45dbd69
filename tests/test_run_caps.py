"""Which LDS cap a tuned run takes, checked on the CPU with the HIP calls of the host
runtime answered by the test."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, os.path.join(ROOT, "paper_2001_09761_amd"))


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="hipcc not installed")
def test_plain_cap_is_for_runs_of_one_event(tmp_path):
    import build as B
    flags = [f for f in B.FLAGS if f not in ("-shared", "-fPIC", "-O3")]
    exe = str(tmp_path / "run_caps")
    cmd = [B.HIPCC, *flags, "-O1", "-I", os.path.join(ROOT, "include"), "-I", B.CSRC,
           os.path.join(ROOT, "tests", "host_checks", "run_caps.hip"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
