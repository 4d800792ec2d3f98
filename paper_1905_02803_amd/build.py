"""Build the HIP library libpencilfft.so in-tree for gfx950 with hipcc.

Usage: python -m paper_1905_02803_amd.build   (or build() from Python).
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libpencilfft.so")
# the mixed-radix kernels: one source, compiled once per unit and precision
MR_UNITS = 8
MR_PARTS = {f"kernels_mr_{t}_{u}.hip": [f"-DPF_MR_UNIT={u}", f"-DPF_MR_UNITS={MR_UNITS}", f"-DPF_MR_T={t}",
                                        f"-DPF_MR_NAME=mr_pick_{t}_{u}"]
            for t in ("double", "float") for u in range(MR_UNITS)}
MR_CLASSES = 6  # classes of lengths with a batched kernel (kernels_mr.h, kMrClass)
MR_PARTS.update({f"kernels_mr_class_{t}_{c}.hip": [f"-DPF_MR_CLASS={c}", f"-DPF_MR_T={t}",
                                                   f"-DPF_MR_NAME=mr_class_{t}_{c}"]
                 for t in ("double", "float") for c in range(MR_CLASSES)})
# object names (with .hip in place of .o), the slowest to compile first
SOURCES = ["kernels_p2.hip", *MR_PARTS, "capi.hip", "kernels.hip", "kernels_mr.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    # keep the compiler from forming packed FP32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def build(verbose: bool = False, out: str = LIB, extra=()) -> str:
    """Compile every source to an object, link the shared library, return its path."""
    objs = []
    bdir = os.path.join(os.path.dirname(out), "_build")
    os.makedirs(bdir, exist_ok=True)
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    cmds = []
    for src in SOURCES:
        obj = os.path.join(bdir, src.replace(".hip", ".o"))
        path = os.path.join(CSRC, src if src not in MR_PARTS else
                            "kernels_mr_class.hip" if "_class_" in src else "kernels_mr_unit.hip")
        cmds.append([HIPCC] + FLAGS + list(extra) + MR_PARTS.get(src, []) + inc + ["-c", path, "-o", obj])
        if verbose:
            print(" ".join(cmds[-1]), flush=True)
        objs.append(obj)
    # the sources compile concurrently, as many at a time as there are CPUs to run them
    with ThreadPoolExecutor(max(1, min(16, len(os.sched_getaffinity(0))))) as ex:
        codes = list(ex.map(lambda c: subprocess.run(c).returncode, cmds))
    failed = [cmd for code, cmd in zip(codes, cmds) if code != 0]
    if failed:
        raise subprocess.CalledProcessError(1, failed[0])
    tmp = out + ".tmp%d" % os.getpid()
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, out)
    return out


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
