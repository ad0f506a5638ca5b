"""Build the gfx950 shared library libstlmi.so in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libstlmi.so")
SOURCES = ["stl_exec_bwd.hip", "stl_exec_bwd_ws.hip", "stl_exec_fwd.hip", "stl_kernels.hip", "mlp_kernels.hip",
           "stl_api.cpp", "stl_compile.cpp"]
ARCH = "gfx950"

HIPCC_FLAGS = [
    "--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC",
    # packed fp32 ops off: hipcc may emit them by itself otherwise
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def build(verbose: bool = False) -> str:
    """Compile every source (in parallel) and link libstlmi.so; always recompiles."""
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    tmp = LIB + ".tmp%d" % os.getpid()

    def run(cmd):
        r = subprocess.run([hipcc] + cmd, capture_output=True, text=True)
        if r.returncode != 0:
            sys.stderr.write(r.stdout + r.stderr)
            raise RuntimeError("hipcc failed building libstlmi.so")
        if verbose:
            sys.stderr.write(r.stderr)

    with tempfile.TemporaryDirectory() as d:
        objs = [os.path.join(d, s + ".o") for s in SOURCES]
        jobs = [HIPCC_FLAGS + ["-c", os.path.join(CSRC, s), "-o", o] for s, o in zip(SOURCES, objs)]
        with ThreadPoolExecutor(max_workers=4) as ex:
            list(ex.map(run, jobs))
        run(["--offload-arch=" + ARCH, "-shared", "-fPIC"] + objs + ["-o", tmp])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
