"""Build the gfx950 engine library in-tree: paper_2408_00836_amd/libhubvqe.so.

Run as `python -m paper_2408_00836_amd.build` or via __graft_entry__.build().
hipcc cross-compiles for gfx950 without a GPU present.
"""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libhubvqe.so")
SOURCES = ["model.cpp", "plan.cpp", "tridiag.cpp", "lbfgs.cpp", "sector_plan.cpp", "engine.hip",
           "kernels.hip", "ham.hip", "sector.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"


def build(verbose: bool = False) -> str:
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-shared",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           # keep SimplifyCFG from merging the per-register-pair code of the
           # pass kernels into one block with phi'd addresses, which would
           # force the register tiles into scratch memory
           "-mllvm", "-simplifycfg-sink-common=false",
           "-Wall", "-Wno-unused-parameter", "-x", "hip"]
    cmd += [os.path.join(CSRC, s) for s in SOURCES]
    cmd += ["-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass does not know the packed-fp32 feature flag: harmless notice
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed ({res.returncode}):\n{err}")
    if err.strip() and verbose:
        print(err, file=sys.stderr)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
