"""Build the HIP library ``_lib/libng.so`` for gfx950 with hipcc.

Flags: -O3; no multiply-add contraction (-ffp-contract=off; the FP32 kernels
write their fused multiply-adds explicitly, the FP64 kernels follow the plain
evaluation order of the formulas); packed FP32 instructions disabled.
"""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "_lib", "libng.so")
SOURCES = ["ng_kernels.hip", "ng_resident.hip", "ng_resident2d.hip", "ng_api.cpp"]
ARCH = os.environ.get("NG_OFFLOAD_ARCH", "gfx950")

FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def build(verbose: bool = False) -> str:
    """Compile the sources (in parallel, one hipcc each) and link them."""
    os.makedirs(os.path.dirname(OUT), exist_ok=True)
    with tempfile.TemporaryDirectory(dir=os.path.dirname(OUT)) as tmp:
        objs = [os.path.join(tmp, s + ".o") for s in SOURCES]
        jobs = [subprocess.Popen(["hipcc", *FLAGS, "-c", "-o", o, os.path.join(CSRC, s)],
                                 stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
                for s, o in zip(SOURCES, objs)]
        said = [j.communicate()[0] for j in jobs]
        if any(j.returncode for j in jobs):
            sys.stderr.write("".join(said))
            raise RuntimeError("hipcc failed")
        lib = os.path.join(tmp, "libng.so")
        r = subprocess.run(["hipcc", *FLAGS, "-shared", "-o", lib, *objs], capture_output=True,
                           text=True)
        if r.returncode != 0:
            sys.stderr.write(r.stdout + r.stderr)
            raise RuntimeError("hipcc failed")
        if verbose:
            sys.stderr.write("".join(said) + r.stderr)
        os.replace(lib, OUT)
    return OUT


if __name__ == "__main__":
    print(build(verbose=True))
