"""Build script of libflipmc.so (hipcc, gfx950)."""
from __future__ import annotations

import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SOURCES = [os.path.join(HERE, "csrc", f) for f in ("kernels.hip", "capi.hip", "flex.hip")]
OUT = os.path.join(HERE, "libflipmc.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # contraction only where the code asks for fma(): proposals, wraps and
    # cell indices then round exactly like the FP64 reference definitions
    "-ffp-contract=off",
    # no packed FP32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


# The rigid engine's sweep kernels are one loop around all of a sweep's work:
# hoisting the constants of every part out of it fills the registers, and each
# colour then reloads a hundred spilled values (1728 molecules on one workgroup:
# 594 us a sweep with it, 565 without).  The flexible engine's are 10 % slower
# without it.
FILE_FLAGS = {"kernels.hip": ["-mllvm", "-disable-machine-licm"]}

# roctx ranges of the host API calls (rocprofv3 --marker-trace)
LINK_FLAGS = ["-lrocprofiler-sdk-roctx"]


def _run(cmd):
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + res.stderr[-4000:])


def build(verbose: bool = False) -> str:
    with tempfile.TemporaryDirectory() as tmp, ThreadPoolExecutor(len(SOURCES)) as pool:
        objects, cmds = [], []
        for src in SOURCES:
            name = os.path.basename(src)
            objects.append(os.path.join(tmp, name + ".o"))
            cmds.append(["hipcc", *(f for f in HIPCC_FLAGS if f != "-shared"), *FILE_FLAGS.get(name, []), "-I" + os.path.join(ROOT, "include"),
                         "-c", src, "-o", objects[-1]])
        link = ["hipcc", "--offload-arch=gfx950", "-shared", *objects, "-o", OUT, *LINK_FLAGS]
        if verbose:
            print("\n".join(" ".join(c) for c in [*cmds, link]), flush=True)
        list(pool.map(_run, cmds))
        _run(link)
    return OUT


if __name__ == "__main__":
    print(build(verbose=True))
