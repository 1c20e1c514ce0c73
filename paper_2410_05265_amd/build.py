"""Builds libpq.so (the HIP kernels and their C ABI) in-tree for gfx950 with hipcc, and the binding's native call path with g++."""

from __future__ import annotations

import concurrent.futures
import glob
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ_DIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libpq.so")
CALL_SRC = os.path.join(CSRC, "pq_call.cpp")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# packed fp32 VALU forms are switched off on purpose (they are not trusted on the test machines)
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _newest_dep():
    deps = sources() + glob.glob(os.path.join(CSRC, "*.h")) + [os.path.join(HERE, "..", "include", "pq.h")]
    return max(os.path.getmtime(d) for d in deps)


def _older(path, time) -> bool:
    return not os.path.exists(path) or os.path.getmtime(path) < time


def _call_path():
    """Where the native call path belongs: named after this Python and this torch, so a build for others does not count; None without torch."""
    try:
        from .binding import CALL_PATH
    except ImportError:
        return None
    return CALL_PATH


def _call_is_stale() -> bool:
    path = _call_path()
    return path is not None and _older(path, os.path.getmtime(CALL_SRC))


def is_stale() -> bool:
    return _older(LIB, _newest_dep()) or _call_is_stale()


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, os.path.basename(src) + ".o")
    subprocess.run([HIPCC, *FLAGS, "-c", src, "-o", obj], check=True)
    return obj


def _build_call() -> bool:
    """Whether the native call path could be built: it needs g++ and the headers of torch and Python, and every call works without it."""
    path = _call_path()
    if path is None:
        return False
    import torch
    root = os.path.dirname(torch.__file__)
    tmp = path + ".tmp%d" % os.getpid()
    try:
        subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
                        "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
                        *("-isystem" + d for d in (root + "/include", root + "/include/torch/csrc/api/include", "/opt/rocm/include",
                                                   sysconfig.get_paths()["include"])),
                        CALL_SRC, "-o", tmp, "-L" + root + "/lib", "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"], check=True)
    except (OSError, subprocess.CalledProcessError) as e:
        print("the native call path was not built, calls will go through ctypes: %s" % e, file=sys.stderr)
        return False
    os.replace(tmp, path)
    return True


def build_lib(force: bool = True, verbose: bool = False) -> str:
    """Compile every .hip source and link libpq.so; returns its path."""
    if not force and not _older(LIB, _newest_dep()):
        if _call_is_stale():
            _build_call()
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
