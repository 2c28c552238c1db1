"""Builds librespec.so (HIP, gfx950 only) in-tree with hipcc.

    python -m paper_2510_26475_amd.build        # compile if sources are newer
    python -m paper_2510_26475_amd.build -f     # always compile
"""
from __future__ import annotations

import os
import subprocess
import sys

_HERE = os.path.dirname(os.path.abspath(__file__))
_ROOT = os.path.dirname(_HERE)
CSRC = os.path.join(_HERE, "csrc")
INCLUDE = os.path.join(_ROOT, "include")
LIB_PATH = os.path.join(_HERE, "librespec.so")

SOURCES = ["respec_common.hip", "respec_solver.hip", "respec_validate.hip", "respec_sampler.hip", "respec_tree_sampler.hip", "respec_kd.hip",
           "respec_attention.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed fp32 VALU forms are kept off: some have given wrong results here
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    f"-I{INCLUDE}", f"-I{CSRC}",
]


def _inputs():
    files = [os.path.join(CSRC, s) for s in SOURCES]
    files += [os.path.join(CSRC, "respec_common.hpp"), os.path.join(CSRC, "respec_sampler_rows.hpp"),
              os.path.join(CSRC, "respec_sampler_share.hpp"), os.path.join(CSRC, "respec_tree_candidate.hpp"),
              os.path.join(CSRC, "respec_kd_absent.hpp"), os.path.join(INCLUDE, "respec.h")]
    return files


def needs_build() -> bool:
    if not os.path.exists(LIB_PATH):
        return True
    t = os.path.getmtime(LIB_PATH)
    return any(os.path.getmtime(f) > t for f in _inputs())


def build(force: bool = False, verbose: bool = False) -> str:
    if not force and not needs_build():
        return LIB_PATH
    cmd = [HIPCC] + FLAGS + [os.path.join(CSRC, s) for s in SOURCES] + ["-o", LIB_PATH]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed ({res.returncode}):\n{err}")
    if verbose and err.strip():
        print(err, flush=True)
    return LIB_PATH


if __name__ == "__main__":
    build(force="-f" in sys.argv[1:], verbose=True)
    print(LIB_PATH)
