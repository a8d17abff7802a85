"""Host-side checks of the halved columns' geometry and index maps (CPU only):
see tests/host_index/pair_halves.cpp."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None and not os.path.exists(HIPCC), reason="hipcc not available")
def test_halved_columns_geometry_and_maps(tmp_path):
    exe = tmp_path / "pair_halves"
    src = os.path.join(ROOT, "tests", "host_index", "pair_halves.cpp")
    r = subprocess.run([HIPCC, "-std=c++17", "-O1", "-x", "hip", "--offload-host-only",
                        "-I", os.path.join(ROOT, "paper_1304_2062_amd", "csrc"), src, "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    m = re.search(r"plans (\d+) bad 0", r.stdout)
    assert m and int(m.group(1)) > 0, r.stdout
