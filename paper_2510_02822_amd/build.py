"""Builds libflexiq.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libflexiq.so")
# Python's way into the run-time entry points (csrc/calls.cpp), for this Python and this torch
CALLS = os.path.join(HERE, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))
NUM_TILE_SHAPES = 15
# (source, object, extra flags): the kernel of every tile shape is a translation unit of its own
UNITS = [("pack.hip", "pack.o", []), ("gemm.hip", "gemm.o", []), ("fp6_gemm.hip", "fp6_gemm.o", []),
         ("smallm.hip", "smallm.o", []), ("stream.hip", "stream.o", []), ("conv3.hip", "conv3.o", []),
         ("halo.hip", "halo.o", []), ("wreg.hip", "wreg.o", []), ("wreg6.hip", "wreg6.o", []), ("chunk.hip", "chunk.o", [])] + \
        [("mixed_tile.hip", "mixed_tile_%d.o" % i, ["-DFQ_TILE=%d" % i]) for i in range(NUM_TILE_SHAPES)]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function", "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def _calls_command():
    import torch
    T = os.path.dirname(torch.__file__)
    inc = [os.path.join(T, "include"), os.path.join(T, "include", "torch", "csrc", "api", "include"), sysconfig.get_paths()["include"],
           os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), os.path.join(ROOT, "include")]
    return ["g++", "-std=c++17", "-O2", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-Wno-unused-function", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
            "-DBUILT_FOR=\"%s\"" % torch.__version__,
            "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), *sum((["-isystem", i] for i in inc[:-1]), []), "-I", inc[-1],
            os.path.join(CSRC, "calls.cpp"), "-o", CALLS, "-L", os.path.join(T, "lib"), "-lc10", "-ltorch_cpu", "-lc10_hip", "-ltorch_python"]


def _start(cmd):
    return cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)


def _finish(job, verbose: bool):
    """Raises if the command failed."""
    cmd, pr = job
    out, _ = pr.communicate()
    out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
    if pr.returncode != 0:
        raise RuntimeError("%s failed: %s\n%s" % (os.path.basename(cmd[0]), " ".join(cmd), out))
    if verbose and out.strip():
        print(out)


def build(verbose: bool = False, extra=()) -> str:
    """Builds the library, and the native calls where torch's and Python's headers and a C++ compiler are there (the Python functions
    behind them serve every call without)."""
    calls, why = None, None
    try:
        calls = _start(_calls_command())
    except (ImportError, OSError) as e:
        why = e
    jobs = [_start(["hipcc", *FLAGS, *defs, *extra, "-c", os.path.join(CSRC, src), "-o", os.path.join(CSRC, o)]) for src, o, defs in UNITS]
    if calls:
        try:
            _finish(calls, verbose)
        except RuntimeError as e:
            why = e
    if why is not None:
        print("the native calls were not built: %s" % why, file=sys.stderr)
        if os.path.exists(CALLS):   # (of other sources)
            os.remove(CALLS)
    for job in jobs:
        _finish(job, verbose)
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *[os.path.join(CSRC, o) for _, o, _ in UNITS]])
    return LIB


if __name__ == "__main__":
    print(build(verbose=True, extra=sys.argv[1:]))
