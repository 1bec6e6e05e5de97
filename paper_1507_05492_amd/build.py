"""Build step: compile the HIP sources into ``libcq.so`` (gfx950) next to this file.

``python paper_1507_05492_amd/build.py`` or :func:`build` (load this file by path:
importing it through the package runs the package's ``__init__``, which loads the
library).  hipcc cross-compiles for gfx950 without a GPU present.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRC = os.path.join(HERE, "csrc", "cq_lib.hip")
DEPS = [os.path.join(HERE, "csrc", f) for f in ("cq_device.hpp", "cq_kernels.hpp", "cq_compare.hpp", "cq_rows.hpp", "cq_small.hpp", "cq_tiles.hpp", "srv_core.hpp")] + [os.path.join(ROOT, "include", "cq.h")]
OUT = os.path.join(HERE, "libcq.so")
ARCH = "gfx950"


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (ROCm is required to build the library)")


def command(out: str = OUT) -> list[str]:
    return [
        hipcc(), f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-shared",
        # packed fp32 instructions are kept out of the generated code
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        "-I", os.path.join(ROOT, "include"), "-I", os.path.join(HERE, "csrc"),
        SRC, "-o", out,
    ]


def build(verbose: bool = False) -> str:
    tmp = OUT + ".tmp"
    cmd = command(tmp)
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("hipcc failed")
    os.replace(tmp, OUT)
    return OUT


def stale() -> bool:
    if not os.path.exists(OUT):
        return True
    t = os.path.getmtime(OUT)
    return any(os.path.getmtime(p) > t for p in [SRC] + DEPS)


if __name__ == "__main__":
    print(build(verbose=True))
