"""Builds libesp.so (HIP, gfx950 only, hipcc) and the binding's argument checks (g++) in-tree.  No GPU is needed to build."""
from __future__ import annotations

import glob
import os
import shutil
import subprocess
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
LIB = os.path.join(PKG, "libesp.so")
SOURCES = sorted(glob.glob(os.path.join(PKG, "csrc", "*.hip")))
HEADERS = sorted(glob.glob(os.path.join(PKG, "csrc", "*.h"))) + [os.path.join(ROOT, "include", "esp.h")]

MARSHAL_SOURCE = os.path.join(PKG, "csrc", "marshal.cpp")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-shared",
    # packed-fp32 VALU forms are kept out of the generated code on the test machines
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the first arguments of a kernel are in scalar registers when its wavefronts start, not a round trip away (only plain ones that come
    # first, no structs): decode steps, us: 16 requests of 900, 32 / 8 heads, 19.4 -> 18.9, 40 of 150, 40 / 8, 17.1 -> 16.6, 34 of 78, 12 / 12, 17.2 -> 16.6
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-I" + os.path.join(ROOT, "include"),
]


def marshal_path() -> str:
    """The native argument checks unpack torch's and Python's own objects: the file is named after those that it is built for, so that
    after a change of either it is not found (and built again) rather than loaded."""
    import torch
    return os.path.join(PKG, f"_marshal.torch-{torch.__version__}-abi{int(torch._C._GLIBCXX_USE_CXX11_ABI)}{sysconfig.get_config_var('EXT_SUFFIX')}")


def _older(built: str, sources) -> bool:
    return not os.path.exists(built) or any(os.path.getmtime(f) > os.path.getmtime(built) for f in sources)


def is_stale() -> bool:
    """Built before its sources, or before this file, which has the flags."""
    if _older(LIB, SOURCES + HEADERS + [__file__]):
        return True
    return shutil.which("g++") is not None and _older(marshal_path(), [MARSHAL_SOURCE, os.path.join(ROOT, "include", "esp.h"), __file__])


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
    if shutil.which("g++") is not None:
        build_marshal()
    else:
        print("g++ is missing: the binding's native argument checks are not built, its Python checks are used alone")
    return LIB


def build_marshal() -> str:
    """Compile the native argument checks against the installed torch.  Returns the module's path."""
    import torch
    base, path = os.path.dirname(torch.__file__), marshal_path()
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-w",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(base, "include"),
           "-I" + os.path.join(base, "include", "torch", "csrc", "api", "include"), "-I" + sysconfig.get_paths()["include"],
           MARSHAL_SOURCE, "-o", path, "-L" + os.path.join(base, "lib"), "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10",
           "-Wl,-rpath," + os.path.join(base, "lib")]
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if proc.returncode != 0:
        raise RuntimeError("g++ failed:\n" + proc.stdout)
    return path


if __name__ == "__main__":
    print(build_lib(force=True, verbose=True))
