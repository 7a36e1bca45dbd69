"""The unit path's arrays lie at the ends of buffers that the general path also
uses: within one launch no workgroup may write what another still reads. Checked
on the CPU over the sizes the path takes (a workgroup that starts late must find
the verdict as k_units left it, also where the others have gone on to the general
path's histogram)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, os.path.join(ROOT, "paper_2001_09761_amd"))


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="hipcc not installed")
def test_unit_arrays_are_disjoint_from_what_the_launch_writes(tmp_path):
    import build as B
    flags = [f for f in B.FLAGS if f not in ("-shared", "-fPIC", "-O3")]
    exe = str(tmp_path / "unit_layout")
    cmd = [B.HIPCC, *flags, "-O1", "-I", os.path.join(ROOT, "include"), "-I", B.CSRC,
           os.path.join(ROOT, "tests", "host_checks", "unit_layout.hip"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
