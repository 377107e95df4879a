"""Builds the gfx950 shared library (csrc/*.hip -> libla_hip.so) with hipcc, and the binding's
native argument checks (csrc/la_call.cpp -> _call.so) with g++.

hipcc cross-compiles without a GPU, so this runs anywhere the ROCm toolchain is
installed.  The library is kept in-tree next to this file.  It needs neither torch nor Python;
_call.so needs the headers of both and is left out where they, or g++, are missing: the binding
then makes the same calls through its Python checks.
"""
from __future__ import annotations

import concurrent.futures
import glob
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(CSRC, "_build")
LIB = os.path.join(HERE, "libla_hip.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


CALL = os.path.join(HERE, "_call.so")


def _call_command():
    """The command that builds _call.so, or None where its headers or its compiler are missing."""
    import sysconfig
    try:
        import torch
    except ImportError:
        return None
    root, python = os.path.dirname(torch.__file__), sysconfig.get_paths()["include"]
    needed = (os.path.join(root, "include", "torch", "csrc", "autograd", "python_variable.h"),
              os.path.join(root, "include", "c10", "hip", "HIPStream.h"), os.path.join(python, "Python.h"))
    if shutil.which("g++") is None or not all(os.path.exists(f) for f in needed):
        return None
    return ["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            "-isystem", os.path.join(root, "include"), "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"),
            "-isystem", "/opt/rocm/include", "-isystem", python, os.path.join(CSRC, "la_call.cpp"), "-o", CALL,
            "-L", os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip",
            f"-Wl,-rpath,{os.path.join(root, 'lib')}"]


def _build_call() -> None:
    """The native argument checks (csrc/la_call.cpp), a CPython module on torch's headers; host code."""
    command = _call_command()
    if command is None:
        if os.path.exists(CALL):             # of older sources
            os.remove(CALL)
        print("_call.so left out: torch's or Python's headers or g++ not found", file=sys.stderr)
        return
    subprocess.run(command, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _deps_mtime():
    files = sources() + glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.cpp")) + \
        glob.glob(os.path.join(HERE, "..", "include", "*.h"))
    return max(os.path.getmtime(f) for f in files)


def is_current() -> bool:
    files = (LIB, CALL) if _call_command() is not None else (LIB,)
    return all(os.path.exists(f) and os.path.getmtime(f) >= _deps_mtime() for f in files)


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.basename(src)[:-4] + ".o")
    subprocess.run([HIPCC, *FLAGS, "-c", src, "-o", obj], check=True, cwd=CSRC,
                   stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    return obj


def build_library(force: bool = True, jobs: int = 6) -> str:
    """Compile every HIP source for gfx950, link libla_hip.so, and build _call.so where that can be.  With
    force=False an up-to-date library is left alone."""
    if not force and is_current():
        return LIB
    os.makedirs(OBJ, exist_ok=True)
    try:
        with concurrent.futures.ThreadPoolExecutor(max_workers=jobs) as ex:
            call = ex.submit(_build_call)
            objs = list(ex.map(_compile, sources()))
            call.result()
        subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs],
                       check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    except subprocess.CalledProcessError as e:  # show the compiler's message
        raise RuntimeError(f"{e.cmd[0]} failed:\n{e.stdout.decode(errors='replace')}") from e
    return LIB


if __name__ == "__main__":
    print(build_library(force=True))
