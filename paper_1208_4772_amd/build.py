"""Build ``libdg.so`` (HIP for gfx950) in-tree with hipcc.

Usage: ``python -m paper_1208_4772_amd.build`` or :func:`build`.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdg.so")
SOURCES = ["kernels.hip", "stage_mfma.hip", "stage64.hip", "weak.hip", "tet3d.hip", "api.cpp", "api3.cpp",
           "refelem.cpp"]
ARCH = os.environ.get("DG_OFFLOAD_ARCH", "gfx950")

# Packed FP32 instructions stay disabled; hipcc's host pass warns that it
# does not know the feature, which is harmless.  Multiply-adds are fused only
# within one source expression (-ffp-contract=on), so the rounding of every
# result is fixed by the source: the single-mesh and the batched kernels,
# built from the same code, give the same bits.
HIP_FLAGS = ["-O3", "-std=c++17", "-fPIC", "-ffp-contract=on", f"--offload-arch={ARCH}",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-Wno-unused-command-line-argument", "-Wno-pass-failed"]


def hipcc() -> str:
    for cand in (os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc"),
                 shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def build(verbose: bool = False) -> str:
    """Compile every source and link ``libdg.so``; returns its path."""
    cc = hipcc()
    tmp = tempfile.mkdtemp(prefix="dgbuild_")
    try:
        def compile_one(src):
            obj = os.path.join(tmp, os.path.splitext(src)[0] + ".o")
            cmd = [cc, "-x", "hip", *HIP_FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            r = subprocess.run(cmd, capture_output=True, text=True)
            if r.returncode != 0:
                raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr}")
            return obj
        with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
            objs = list(ex.map(compile_one, SOURCES))
        out_tmp = LIB + f".tmp{os.getpid()}"
        cmd = [cc, "-shared", f"--offload-arch={ARCH}", *objs, "-o", out_tmp]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"link failed:\n{r.stderr}")
        os.replace(out_tmp, LIB)
    finally:
        shutil.rmtree(tmp, ignore_errors=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
