"""The kernels of the unit path and of the all-pairs form compile for gfx950 with no
scratch at all: their compiler reports, built here on the CPU."""
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, os.path.join(ROOT, "paper_2001_09761_amd"))


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="hipcc not installed")
@pytest.mark.parametrize("source,at_least", [("clue_units.hip", 6), ("clue_direct.hip", 11)])
def test_no_scratch(source, at_least, tmp_path):
    import build as B
    flags = [f for f in B.FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [B.HIPCC, *flags, "-I", os.path.join(ROOT, "include"), "-I", B.CSRC, "-c", os.path.join(B.CSRC, source),
           "-o", str(tmp_path / "k.o"), "-Rpass-analysis=kernel-resource-usage"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    sizes = [int(v) for v in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)]
    report = {n: s for n, s in zip(names, sizes) if "k_" in n}
    assert len(names) == len(sizes) and len(report) >= at_least, names
    assert not any(report.values()), report
