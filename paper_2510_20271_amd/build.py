"""Compile the HIP sources into ``paper_2510_20271_amd/libecc_hip.so`` (gfx950).

Every source file is compiled to an object of its own (in parallel, into ``_build/`` next to
this file) and the objects are linked into the shared library.  The layer's autograd function
(``csrc/layer_torch.cpp``) is a torch extension, ``_layer_native.so``, linked against that library.
"""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SO = os.path.join(HERE, "libecc_hip.so")
OBJ_DIR = os.path.join(HERE, "_build")
LAYER_SO = os.path.join(HERE, "_layer_native.so")
SOURCES = sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip")))
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def build_library(verbose: bool = False, extra=()) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ_DIR, exist_ok=True)

    def compile_one(src: str) -> str:
        obj = os.path.join(OBJ_DIR, os.path.basename(src)[:-4] + ".o")
        cmd = [hipcc, *FLAGS, *extra, "-I", os.path.join(ROOT, "include"), "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        return obj

    with ThreadPoolExecutor(max_workers=8) as pool:
        layer = pool.submit(compile_layer, verbose)
        objects = list(pool.map(compile_one, SOURCES))
        layer_obj = layer.result()
    link = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", SO, *objects]
    if verbose:
        print(" ".join(link), flush=True)
    subprocess.check_call(link)
    link_layer(layer_obj, verbose)
    return SO


def compile_layer(verbose: bool = False) -> str:
    from torch.utils import cpp_extension
    obj = os.path.join(OBJ_DIR, "layer_torch.o")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1",
           "-DUSE_ROCM=1", "-DTORCH_EXTENSION_NAME=_layer_native", "-DTORCH_API_INCLUDE_EXTENSION_H"]
    for path in cpp_extension.include_paths("cuda") + [sysconfig.get_path("include"), os.path.join(ROOT, "include")]:
        cmd += ["-isystem" if path != os.path.join(ROOT, "include") else "-I", path]
    cmd += ["-c", os.path.join(HERE, "csrc", "layer_torch.cpp"), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return obj


def link_layer(obj: str, verbose: bool = False) -> str:
    from torch.utils import cpp_extension
    cmd = [os.environ.get("CXX", "g++"), "-shared", "-o", LAYER_SO, obj, "-L", HERE, "-l:libecc_hip.so", "-Wl,-rpath,$ORIGIN"]
    for path in cpp_extension.library_paths("cuda"):
        cmd += ["-L", path]
    cmd += ["-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return LAYER_SO


if __name__ == "__main__":
    build_library(verbose=True, extra=sys.argv[1:])
