"""Build libsrmd.so (HIP, gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libsrmd.so")
# one translation unit each: the kernels once per threads-per-particle value (compiled
# side by side), everything else once
UNITS = [("kernels.hip", f"-DSRMD_TP={tp}") for tp in (1, 2, 4, 8, 16, 32, 64)] + [("kernels.hip", ""), ("runtime.hip", "")]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # parity-critical float32 arithmetic: no contraction, no fast math
    "-ffp-contract=off", "-fno-fast-math",
    # no compiler-generated packed fp32 ops
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result", "-Wno-unused-function", "-Wno-unused-const-variable",
]


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB + ".tmp"

    def run(cmd):
        res = subprocess.run(cmd, capture_output=True, text=True)
        err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + " ".join(cmd) + "\n" + err)
        if verbose and err.strip():
            print(err, file=sys.stderr)

    with tempfile.TemporaryDirectory(prefix="srmd_build_") as objs:
        def compile_unit(k):
            src, define = UNITS[k]
            obj = os.path.join(objs, f"{k}.o")
            run([hipcc, *HIPCC_FLAGS, *([define] if define else []), "-c", "-I", os.path.join(ROOT, "include"), "-o", obj,
                 os.path.join(CSRC, src)])
            return obj

        with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
            files = list(pool.map(compile_unit, range(len(UNITS))))
        run([hipcc, "--offload-arch=gfx950", "-fPIC", "-shared", "-o", tmp, *files])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
