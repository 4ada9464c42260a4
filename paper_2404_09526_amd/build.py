"""Builds libesp.so (HIP, gfx950 only, hipcc) and the binding's argument checks (_marshal.so, g++) in-tree.  No GPU is needed to build."""
from __future__ import annotations

import glob
import os
import subprocess

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
LIB = os.path.join(PKG, "libesp.so")
SOURCES = sorted(glob.glob(os.path.join(PKG, "csrc", "*.hip")))
HEADERS = sorted(glob.glob(os.path.join(PKG, "csrc", "*.h"))) + [os.path.join(ROOT, "include", "esp.h")]

MARSHAL = os.path.join(PKG, "_marshal.so")
MARSHAL_SOURCE = os.path.join(PKG, "csrc", "marshal.cpp")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-shared",
    # packed-fp32 VALU forms are kept out of the generated code on the test machines
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + os.path.join(ROOT, "include"),
]


def is_stale() -> bool:
    for built, sources in ((LIB, SOURCES + HEADERS), (MARSHAL, [MARSHAL_SOURCE, os.path.join(ROOT, "include", "esp.h")])):
        if not os.path.exists(built) or any(os.path.getmtime(f) > os.path.getmtime(built) for f in sources):
            return True
    return False


def build_lib(force: bool = True, verbose: bool = False) -> str:
    """Compile every HIP source into libesp.so, and the binding's argument checks.  Returns the library path."""
    if not force and not is_stale():
        return LIB
    cmd = [HIPCC] + FLAGS + SOURCES + ["-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in proc.stdout.splitlines() if "not a recognized feature" not in l)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)
    build_marshal()
    return LIB


def build_marshal() -> str:
    """Compile the native argument checks against the installed torch.  Returns the module's path."""
    import sysconfig
    import torch
    base = os.path.dirname(torch.__file__)
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-w",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(base, "include"),
           "-I" + os.path.join(base, "include", "torch", "csrc", "api", "include"), "-I" + sysconfig.get_paths()["include"],
           MARSHAL_SOURCE, "-o", MARSHAL, "-L" + os.path.join(base, "lib"), "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10",
           "-Wl,-rpath," + os.path.join(base, "lib")]
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if proc.returncode != 0:
        raise RuntimeError("g++ failed:\n" + proc.stdout)
    return MARSHAL


if __name__ == "__main__":
    print(build_lib(force=True, verbose=True))
