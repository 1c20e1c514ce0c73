"""Builds libpq.so (the HIP kernels and their C ABI) in-tree for gfx950 with hipcc, and the binding's native call path with g++."""

from __future__ import annotations

import concurrent.futures
import glob
import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ_DIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libpq.so")
CALL_SRC = os.path.join(CSRC, "pq_call.cpp")
CALL = os.path.join(HERE, "_pq_call.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# packed fp32 VALU forms are switched off on purpose (they are not trusted on the test machines)
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _newest_dep():
    deps = sources() + [CALL_SRC] + glob.glob(os.path.join(CSRC, "*.h")) + [os.path.join(HERE, "..", "include", "pq.h")]
    return max(os.path.getmtime(d) for d in deps)


def is_stale() -> bool:
    return any(not os.path.exists(f) or os.path.getmtime(f) < _newest_dep() for f in (LIB, CALL))


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, os.path.basename(src) + ".o")
    subprocess.run([HIPCC, *FLAGS, "-c", src, "-o", obj], check=True)
    return obj


def _build_call() -> None:
    import torch
    root = os.path.dirname(torch.__file__)
    tmp = CALL + ".tmp%d" % os.getpid()
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
                    "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
                    *("-isystem" + d for d in (root + "/include", root + "/include/torch/csrc/api/include", "/opt/rocm/include",
                                               sysconfig.get_paths()["include"])),
                    CALL_SRC, "-o", tmp, "-L" + root + "/lib", "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"], check=True)
    os.replace(tmp, CALL)


def build_lib(force: bool = True, verbose: bool = False) -> str:
    """Compile every .hip source and link libpq.so; returns its path."""
    if not force and not is_stale():
        return LIB
    os.makedirs(OBJ_DIR, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=8) as ex:
        call = ex.submit(_build_call)
        objs = list(ex.map(_compile, sources()))
        call.result()
    tmp = LIB + ".tmp%d" % os.getpid()
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs], check=True)
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build_lib(force=True, verbose=True)
