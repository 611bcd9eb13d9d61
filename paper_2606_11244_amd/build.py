"""Build the HIP library libspear.so for gfx950 in-tree.

Usage: python -m paper_2606_11244_amd.build   (or call build()).
The library is written next to this file, so that it ships with the source
tree; nothing is installed.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libspear.so")
CEIL = os.path.join(HERE, "libspear_ceiling.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
# Packed fp32 instructions are kept out of the generated code (the hardware
# has given unreliable results with some of their forms); the host pass warns
# that it does not know the feature, which is harmless.
COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}"]

# the kernel files compile once per code width (SPEAR_WB) and activation dtype
UNITS = tuple((src, f"w{wb}_{'bf16' if bf else 'f16'}",
               [f"--offload-arch={ARCH}", "-x", "hip", f"-DSPEAR_WB={wb}", f"-DSPEAR_BF16_UNIT={bf}"])
              for src in ("spear_kernels.hip", "spear_gemm.hip", "spear_mid.hip") for wb in (4, 3) for bf in (0, 1)) + (
    ("spear_api.cpp", "", [f"--offload-arch={ARCH}", "-x", "hip"]),
    ("spear_sched.cpp", "", [f"--offload-arch={ARCH}"]))


def _run(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("hipcc failed: " + " ".join(cmd))
    return r


def build(verbose: bool = False) -> str:
    """Compile every HIP/C++ source of the library (in parallel processes) and
    link libspear.so. The measured-ceiling kernels go into
    libspear_ceiling.so."""
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    cmds, objs = [], []
    for src, tag, extra in UNITS:
        obj = os.path.join(objdir, src + (("." + tag) if tag else "") + ".o")
        cmd = [HIPCC] + COMMON + extra + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd))
        cmds.append(cmd)
        objs.append(obj)
    with cf.ThreadPoolExecutor(len(cmds)) as ex:
        list(ex.map(_run, cmds))
    tmp = LIB + ".tmp"
    _run([HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp] + objs)
    os.replace(tmp, LIB)
    # the measured-ceiling kernels (measurement only), a library of their own
    tmp = CEIL + ".tmp"
    _run([HIPCC] + COMMON + [f"--offload-arch={ARCH}", "-x", "hip", "-shared",
                             os.path.join(CSRC, "spear_ceiling.hip"), "-o", tmp])
    os.replace(tmp, CEIL)
    shutil.rmtree(objdir, ignore_errors=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
