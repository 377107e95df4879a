"""Builds the gfx950 shared library (csrc/*.hip -> libla_hip.so) with hipcc, and the binding's
native argument checks (csrc/la_call.cpp -> _call.so) with g++.

hipcc cross-compiles without a GPU, so this runs anywhere the ROCm toolchain is
installed.  The library is kept in-tree next to this file.
"""
from __future__ import annotations

import concurrent.futures
import glob
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(CSRC, "_build")
LIB = os.path.join(HERE, "libla_hip.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


CALL = os.path.join(HERE, "_call.so")


def _build_call() -> None:
    """The native argument checks (csrc/la_call.cpp), a CPython module on torch's headers; host code."""
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
                    f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
                    "-I", os.path.join(root, "include"), "-I", os.path.join(root, "include", "torch", "csrc", "api", "include"),
                    "-I", "/opt/rocm/include", "-I", sysconfig.get_paths()["include"],
                    os.path.join(CSRC, "la_call.cpp"), "-o", CALL, "-L", os.path.join(root, "lib"),
                    "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip", f"-Wl,-rpath,{os.path.join(root, 'lib')}"],
                   check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _deps_mtime():
    files = sources() + glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.cpp")) + \
        glob.glob(os.path.join(HERE, "..", "include", "*.h"))
    return max(os.path.getmtime(f) for f in files)


def is_current() -> bool:
    return all(os.path.exists(f) and os.path.getmtime(f) >= _deps_mtime() for f in (LIB, CALL))


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.basename(src)[:-4] + ".o")
    subprocess.run([HIPCC, *FLAGS, "-c", src, "-o", obj], check=True, cwd=CSRC,
                   stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    return obj


def build_library(force: bool = True, jobs: int = 6) -> str:
    """Compile every HIP source for gfx950, link libla_hip.so, and build _call.so.  With
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
        raise RuntimeError(f"hipcc failed:\n{e.stdout.decode(errors='replace')}") from e
    return LIB


if __name__ == "__main__":
    print(build_library(force=True))
