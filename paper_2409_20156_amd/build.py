"""Builds the gfx950 shared library of the package in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "libastra_xc.so")
SOURCES = ["xc_api.hip", "xc_mine.hip", "xc_mine_few.hip", "xc_mine_q8.hip", "xc_sample.hip", "xc_step.hip"]


def build(verbose: bool = False) -> str:
    """Compile every HIP source for gfx950 into libastra_xc.so (always rebuilds)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
           "-I" + os.path.join(ROOT, "include"),
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
    cmd += [os.path.join(CSRC, s) for s in SOURCES]
    cmd += ["-o", LIB_PATH]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if verbose or res.returncode != 0:
        print(res.stdout)
        print(res.stderr)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed with exit code %d" % res.returncode)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
