"""Build libse2n.so (HIP for gfx950) in place, next to this file.

Usage: python -m paper_1304_2062_amd.build   (or call build()).
"""
from __future__ import annotations

import os
import subprocess
import sys
import time

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libse2n.so")
SOURCES = ["se2n_kernels_f32.hip", "se2n_kernels_f64.hip", "se2n_precompute.hip", "se2n_orient.hip", "se2n_solve.hip", "se2n_batch.hip", "se2n_cnn.hip", "se2n_runtime.hip",
           "se2n_batch_host.hip", "se2n_batch_pair.hip", "se2n_pair_rows_f32.hip", "se2n_pair_rows_f64.hip", "se2n_pair_mid_f32.hip", "se2n_pair_mid_f64.hip", "se2n_cnn_host.hip", "se2n_restore.hip", "se2n_solve_iter.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    # no packed FP32 instructions (v_pk_*_f32) anywhere in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def _stale(src: str, obj: str) -> bool:
    if not os.path.exists(obj):
        return True
    deps = [src] + [os.path.join(CSRC, h) for h in os.listdir(CSRC) if h.endswith(".hpp")]
    deps.append(os.path.join(os.path.dirname(HERE), "include", "se2n.h"))
    return any(os.path.getmtime(d) > os.path.getmtime(obj) for d in deps)


def build(verbose: bool = True, force: bool = True) -> str:
    """Compile every HIP source to an object and link the shared library.

    With ``force=False`` objects newer than their sources and headers are reused.
    """
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)
    objs = []
    procs = []
    t0 = time.time()
    for src in SOURCES:
        obj = os.path.join(HERE, "_build", src.replace(".hip", ".o"))
        objs.append(obj)
        if not force and not _stale(os.path.join(CSRC, src), obj):
            continue
        cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
    for src, pr in procs:
        out, _ = pr.communicate()
        text = out.decode(errors="replace")
        # the host pass does not know the device-only feature flag: drop that warning
        text = "\n".join(l for l in text.splitlines() if "packed-fp32-ops" not in l and l.strip())
        if pr.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{text}")
        if verbose and text:
            print(text, file=sys.stderr)
    tmp = LIB + ".tmp%d" % os.getpid()
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs])
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB} in {time.time() - t0:.1f}s", file=sys.stderr)
    return LIB


if __name__ == "__main__":
    build(force="--incremental" not in sys.argv)
