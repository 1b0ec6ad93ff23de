"""Build step: compile the HIP sources under csrc/ into libsqllm.so (gfx950 only) and the Python call path into an extension module of the
interpreter that runs this, in-tree.  The library needs hipcc only; without a C compiler or Python's headers the module is left out, and the
binding calls the library through ctypes."""
from __future__ import annotations

import os
import shlex
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsqllm.so")
PYCALL = os.path.join(HERE, "_pycall" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))   # the name says which interpreter it is for
PYCALL_SOURCE = os.path.join(CSRC, "sqllm_pycall.c")
SOURCES = ["sqllm_kernels.hip", "sqllm_batch.hip", "sqllm_quant.hip", "sqllm_api.cpp"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CC = os.environ.get("CC", "gcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
         # packed-FP32 instructions are kept out of the generated code on purpose
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def sources():
    return [os.path.join(CSRC, s) for s in SOURCES]


def is_stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    headers = [os.path.join(CSRC, h) for h in ("sqllm_kernels.h", "sqllm_decode.h", "sqllm_batch_split.h", "sqllm_csr.h", "sqllm_buckets.h")]
    deps = sources() + headers + [os.path.join(ROOT, "include", "sqllm.h")]
    return any(os.path.getmtime(d) > t for d in deps)


def pycall_is_stale() -> bool:
    return not os.path.exists(PYCALL) or os.path.getmtime(PYCALL_SOURCE) > os.path.getmtime(PYCALL)


def build_pycall() -> str:
    """Compile the extension module; returns its path.  Raises where there is no compiler or no Python.h."""
    part = f"{PYCALL}.{os.getpid()}"
    cmd = shlex.split(CC) + ["-O2", "-Wall", "-shared", "-fPIC", "-I" + sysconfig.get_paths()["include"], PYCALL_SOURCE, "-o", part]
    try:
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError(f"{CC} failed:\n" + res.stdout + res.stderr)
        os.replace(part, PYCALL)                                     # several processes may build it at once
    finally:
        if os.path.exists(part):
            os.remove(part)
    return PYCALL


def build(verbose: bool = False) -> str:
    """Compile unconditionally; returns the path of the shared library."""
    cmd = [HIPCC] + FLAGS + ["-I" + os.path.join(ROOT, "include"), "-I" + CSRC] + sources() + ["-o", LIB]
    res = subprocess.run(cmd, capture_output=True, text=True)
    # hipcc's host pass prints a harmless "unknown target feature" warning for -packed-fp32-ops
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)
    try:
        build_pycall()
    except (OSError, RuntimeError) as e:
        print(f"paper_2306_07629_amd: {os.path.basename(PYCALL)} was not built, calls go through ctypes: {e}", file=sys.stderr, flush=True)
    if verbose:
        print(" ".join(cmd))
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
