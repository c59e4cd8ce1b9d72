"""Build the C-ABI library ``libspinner.so`` from ``csrc/`` with hipcc for gfx950, and the native part of its
binding, ``_native.so``, with the host compiler against torch's headers.

The translation units are compiled in parallel and linked into shared
objects that sit next to this file (in-tree, so they travel with the tree).
"""
from __future__ import annotations

import importlib.util
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libspinner.so")
UNITS = ["api", "fused_none", "fused_cossin", "fused_signbits", "multipass", "hash", "layer", "sketch", "structured", "struct_fft", "struct_fft_13", "struct_fft_14", "blocks", "fused_shared", "fused_begun", "sketch_cols"]
NATIVE = os.path.join(HERE, "_native.so")
CXX = os.environ.get("CXX", "g++")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-I", INCLUDE, "-I", CSRC,
         # packed fp32 VALU forms are not used on this target
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]


def _newer(src_list, target):
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(s) > t for s in src_list)


def build_native(obj: str, verbose: bool = False) -> str:
    """Compile the binding's native part to ``obj`` (a host file: no GPU code)."""
    torch_dir = importlib.util.find_spec("torch").submodule_search_locations[0]
    cmd = [CXX, "-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", "-I", INCLUDE,
           "-isystem", sysconfig.get_paths()["include"], "-isystem", os.path.join(torch_dir, "include"),
           "-isystem", "/opt/rocm/include", "-c", os.path.join(CSRC, "binding_native.cpp"), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("%s failed for binding_native:\n%s" % (CXX, r.stderr[-8000:]))
    return os.path.join(torch_dir, "lib")


def build(force: bool = True, verbose: bool = False, extra_flags=()) -> str:
    os.makedirs(BUILD, exist_ok=True)
    headers = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hpp")]
    headers.append(os.path.join(INCLUDE, "spinner.h"))

    def compile_unit(u):
        src = os.path.join(CSRC, u + ".hip")
        obj = os.path.join(BUILD, u + ".o")
        if force or _newer([src] + headers, obj):
            cmd = [HIPCC, *FLAGS, *extra_flags, "-c", src, "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            r = subprocess.run(cmd, capture_output=True, text=True)
            if r.returncode != 0:
                raise RuntimeError("hipcc failed for %s:\n%s" % (u, r.stderr[-8000:]))
            warn = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip())
            if verbose and warn:
                print(warn, flush=True)
        return obj

    native_obj = os.path.join(BUILD, "binding_native.o")
    with ThreadPoolExecutor(max_workers=min(8, len(UNITS) + 1)) as ex:
        native = ex.submit(build_native, native_obj, verbose)
        objs = list(ex.map(compile_unit, UNITS))
        torch_lib = native.result()
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr[-4000:])
    # torch's libraries are in the process before this module is; the library itself lies beside it
    cmd = [CXX, "-shared", "-o", NATIVE, native_obj, "-L", torch_lib, "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python",
           "-L", HERE, "-lspinner", "-Wl,-rpath,$ORIGIN"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link of the binding failed:\n" + r.stderr[-4000:])
    return LIB


if __name__ == "__main__":
    print(build(force="--incremental" not in sys.argv, verbose=True))
