"""Launch and strip arithmetic of the maps, checked on the host: the header's
host functions compiled by hipcc for the host alone."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no hipcc")
def test_grid_arithmetic_on_the_host(tmp_path):
    exe = str(tmp_path / "grid_checks")
    r = subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17",
                        f"-I{ROOT}/include", f"-I{ROOT}/paper_1609_01490_amd/csrc",
                        os.path.join(ROOT, "tests", "grid_checks.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
