"""Compiles the HIP sources in csrc/ for gfx950 into libtempo.so and the native half of the Python
binding into _native.so (both in-tree, next to this file)."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "libtempo.so")
SOURCES = ("api.hip", "gelu.hip", "layernorm.hip", "attention.hip", "mask.hip", "matmul.hip", "encoder.hip")
NATIVE_PATH = os.path.join(HERE, "_native.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option",
]


def _compile(src: str, obj_dir: str) -> str:
    obj = os.path.join(obj_dir, src.replace(".hip", ".o"))
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr[-6000:]}")
    return obj


def _build_native() -> bool:
    """binding.cpp: host code against torch's headers; finds libtempo.so beside itself.  Needs a host
    compiler and Python's headers, which libtempo.so does not: without them there is no _native.so, not
    even an older one, and the binding makes its calls through ctypes."""
    import torch
    root = os.path.dirname(torch.__file__)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-isystem", os.path.join(root, "include"), "-isystem", "/opt/rocm/include",
           "-isystem", sysconfig.get_paths()["include"],
           os.path.join(CSRC, "binding.cpp"), "-o", NATIVE_PATH, LIB_PATH, "-Wl,-rpath,$ORIGIN",
           "-L", os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    try:
        r = subprocess.run(cmd, capture_output=True, text=True)
        failed, said = r.returncode != 0, r.stderr
    except OSError as e:
        failed, said = True, str(e)
    if said:
        print(f"binding.cpp:\n{said[-6000:]}", file=sys.stderr)
    if failed:
        if os.path.exists(NATIVE_PATH):
            os.remove(NATIVE_PATH)
        print("_native.so was not built: the Python binding makes its calls through ctypes", file=sys.stderr)
    return not failed


def build_library(verbose: bool = True) -> str:
    obj_dir = os.path.join(HERE, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    with ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(lambda s: _compile(s, obj_dir), SOURCES))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-Wl,-soname,libtempo.so", "-o", LIB_PATH, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr[-6000:]}")
    _build_native()
    if verbose:
        print(f"built {LIB_PATH}", file=sys.stderr)
    return LIB_PATH


if __name__ == "__main__":
    build_library()
