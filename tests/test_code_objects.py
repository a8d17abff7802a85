"""Which kernels share a code object of the built library (CPU only).  The first
launch from a code object loads all of it, so a program on the pair path must not
load the five passes with its propagators, nor FP32 work FP64's kernels."""
import glob
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1304_2062_amd", "libse2n.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
KERNEL = re.compile(rb"_ZN4se2n(?:12_GLOBAL__N_1)?\d+(kb?_[a-z0-9_]+?)I?([fd]?)(?:Li|Lb|E)")


@pytest.fixture(scope="module")
def objects(tmp_path_factory):
    """One set of (kernel name, type letter or "") per code object."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("llvm-objdump not available")
    if not os.path.exists(LIB):
        pytest.fail(f"{LIB} is not built (run python -m paper_1304_2062_amd.build)")
    tmp = str(tmp_path_factory.mktemp("objects"))
    shutil.copy(LIB, os.path.join(tmp, "lib.so"))
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp, check=True, capture_output=True)
    found = []
    for f in sorted(glob.glob(os.path.join(tmp, "lib.so.*gfx950*"))):
        with open(f, "rb") as fh:
            found.append({(n.decode(), t.decode()) for n, t in KERNEL.findall(fh.read())})
    return found


def test_propagator_builds_are_alone(objects):
    with_build = [{n for n, _ in o} for o in objects if any(n.startswith("k_precompute") for n, _ in o)]
    assert with_build == [{"k_precompute", "k_precompute_mfma"}]


@pytest.mark.parametrize("kernel", ["k_row_fwd", "k_row_inv", "k_col_fft", "k_col_inv_paired", "k_pair_mid",
                                    "k_pair_fwd", "k_pair_inv"])
def test_types_are_apart(objects, kernel):
    types = [{t for n, t in o if n == kernel} for o in objects if any(n == kernel for n, _ in o)]
    assert sorted(map(sorted, types)) == [["d"], ["f"]]
