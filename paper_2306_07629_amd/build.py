"""Build step: compile the HIP sources under csrc/ into libsqllm.so (gfx950 only) and the Python call path into _pycall.so, in-tree."""
from __future__ import annotations

import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsqllm.so")
PYCALL, PYCALL_SOURCE = os.path.join(HERE, "_pycall.so"), os.path.join(CSRC, "sqllm_pycall.c")
SOURCES = ["sqllm_kernels.hip", "sqllm_batch.hip", "sqllm_quant.hip", "sqllm_api.cpp"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
         # packed-FP32 instructions are kept out of the generated code on purpose
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def sources():
    return [os.path.join(CSRC, s) for s in SOURCES]


def is_stale() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(PYCALL):
        return True
    if os.path.getmtime(PYCALL_SOURCE) > os.path.getmtime(PYCALL):
        return True
    t = os.path.getmtime(LIB)
    headers = [os.path.join(CSRC, h) for h in ("sqllm_kernels.h", "sqllm_decode.h", "sqllm_batch_split.h", "sqllm_csr.h", "sqllm_buckets.h")]
    deps = sources() + headers + [os.path.join(ROOT, "include", "sqllm.h")]
    return any(os.path.getmtime(d) > t for d in deps)


def build(verbose: bool = False) -> str:
    """Compile unconditionally; returns the path of the shared library."""
    cmd = [HIPCC] + FLAGS + ["-I" + os.path.join(ROOT, "include"), "-I" + CSRC] + sources() + ["-o", LIB]
    res = subprocess.run(cmd, capture_output=True, text=True)
    # hipcc's host pass prints a harmless "unknown target feature" warning for -packed-fp32-ops
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)
    res = subprocess.run(["gcc", "-O2", "-Wall", "-shared", "-fPIC", "-I" + sysconfig.get_paths()["include"], PYCALL_SOURCE, "-o", PYCALL], capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("gcc failed:\n" + res.stdout + res.stderr)
    if verbose:
        print(" ".join(cmd))
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
