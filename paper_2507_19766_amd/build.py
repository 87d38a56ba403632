"""Builds libulorl.so (gfx950) in-tree with hipcc, and _marshal.so, the extension module between torch and it, with
the host compiler.  No JIT cache: what is built lives next to the sources so that it travels with the tree."""
from __future__ import annotations

import glob
import os
import subprocess
import sysconfig

_HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(_HERE)
CSRC = os.path.join(_HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB_DIR = os.path.join(_HERE, "lib")
LIB_PATH = os.path.join(LIB_DIR, "libulorl.so")
MARSHAL_PATH = os.path.join(LIB_DIR, "_marshal.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # fused multiply-adds only where the source says fmaf(): the kernels rely on exact
    # rounded products in their error-free transforms
    "-ffp-contract=off",
    # packed-fp32 VALU forms are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _hipcc(args, out_path, verbose):
    tmp = out_path + ".tmp%d" % os.getpid()
    cmd = [HIPCC] + FLAGS + ["-I" + INCLUDE, "-I" + CSRC] + args + ["-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    noise = "is not a recognized feature for this target"
    out = "\n".join(l for l in proc.stdout.splitlines() if noise not in l)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)
    os.replace(tmp, out_path)
    return out_path


def _marshal(verbose):
    """lib/_marshal.so: torch tensors to C arguments; finds libulorl.so beside itself."""
    import torch
    from torch.utils.cpp_extension import include_paths, library_paths

    rocm = os.path.dirname(os.path.dirname(os.path.realpath(HIPCC)))
    system = include_paths() + [sysconfig.get_paths()["include"], os.path.join(rocm, "include"), "/opt/rocm/include"]
    tmp = MARSHAL_PATH + ".tmp%d" % os.getpid()
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-DTORCH_EXTENSION_NAME=_marshal", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, "-I" + INCLUDE]
    for d in system:
        cmd += ["-isystem", d]
    cmd += [os.path.join(CSRC, "torch_marshal.cpp"), "-o", tmp, LIB_PATH, "-Wl,-rpath,$ORIGIN"]
    cmd += ["-L" + d for d in library_paths()]
    cmd += ["-ltorch", "-ltorch_cpu", "-ltorch_python", "-lc10", "-ltorch_hip", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if proc.returncode != 0:
        raise RuntimeError("g++ failed:\n" + proc.stdout)
    os.replace(tmp, MARSHAL_PATH)


def build(verbose: bool = False) -> str:
    """Compile every HIP source (one object each, in parallel), link lib/libulorl.so and build the extension
    module over it; always recompiles."""
    from concurrent.futures import ThreadPoolExecutor

    os.makedirs(LIB_DIR, exist_ok=True)
    obj_dir = os.path.join(LIB_DIR, "obj")
    os.makedirs(obj_dir, exist_ok=True)

    def compile_one(src):
        obj = os.path.join(obj_dir, os.path.basename(src) + ".o")
        return _hipcc(["-c", src], obj, verbose)

    with ThreadPoolExecutor(max_workers=4) as pool:
        objs = list(pool.map(compile_one, sources()))
    _hipcc(["-shared", "-Wl,-soname,libulorl.so"] + objs, LIB_PATH, verbose)
    _marshal(verbose)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
