"""Build libckm.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB_PATH = os.path.join(HERE, "libckm.so")
SOURCES = [os.path.join(HERE, "csrc", "ckm_kernels.hip"), os.path.join(HERE, "csrc", "ckm_plan.hip"),
           os.path.join(HERE, "csrc", "ckm_noalloc.hip"), os.path.join(HERE, "csrc", "ckm_tiles.hip"),
           os.path.join(HERE, "csrc", "ckm_tiles.cpp"),
           os.path.join(HERE, "csrc", "ckm_host.cpp")]
ARCH = "gfx950"


def hipcc_command(out: str) -> list:
    return ["hipcc", "--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC", "-shared",
            "-Wall", "-Wno-unused-result",
            # packed fp32 VALU ops stay off (none are needed; some forms are unreliable)
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-I", os.path.join(ROOT, "include"), "-I", os.path.join(HERE, "csrc"),
            *SOURCES, "-o", out]


def build(verbose: bool = False) -> str:
    tmp = LIB_PATH + ".tmp%d" % os.getpid()
    cmd = hipcc_command(tmp)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("hipcc failed building libckm.so")
    if verbose:
        sys.stderr.write(res.stderr)
    os.replace(tmp, LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
