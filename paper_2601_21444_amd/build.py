"""Build libapbv.so (gfx950) in-tree with hipcc, and the native marshalling of the Python binding (_marshal, an extension of
this interpreter and this torch) with the host compiler where there are torch, its headers and a compiler: the library
works without it.  `python -m paper_2601_21444_amd.build`."""
from __future__ import annotations

import os
import shlex
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libapbv.so")
MARSHAL = os.path.join(PKG, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))
# source -> flags of its own.  The attention kernels: no NaN can arise on their arithmetic paths (masked logits are -inf and
# every inf - inf is guarded), and telling the compiler so drops a canonicalising v_max in front of every maximum.
SOURCES = {
    "api.hip": [],
    "attention.hip": ["-fno-honor-nans"],
    "compress.hip": [],
    "merge.hip": [],
    "packed_attention.hip": ["-fno-honor-nans"],
    "query_attention.hip": ["-fno-honor-nans"],
    "score_matrix.hip": [],
}

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def marshal_commands():
    """Compile and link command of the native marshalling, which calls the libapbv.so beside it; None where it lacks something."""
    cxx = shlex.split(os.environ.get("CXX", "g++"))
    try:
        import torch
        from torch.utils import cpp_extension
        lacks = None if shutil.which(cxx[0]) else f"no compiler {cxx[0]}"
    except ImportError as e:
        lacks = str(e)
    if lacks is None and not os.path.exists(os.path.join(sysconfig.get_paths()["include"], "Python.h")):
        lacks = "no Python.h"
    if lacks is not None:
        print(f"native marshalling not built ({lacks}): the binding goes through ctypes", flush=True)
        return None
    obj = os.path.join(OBJ, "marshal.o")
    includes = [f for p in [*cpp_extension.include_paths(), sysconfig.get_paths()["include"]] for f in ("-isystem", p)]
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    return ([*cxx, "-O2", "-std=c++17", "-fPIC", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *includes,
             "-I", os.path.join(ROOT, "include"), "-c", os.path.join(CSRC, "marshal.cpp"), "-o", obj],
            [*cxx, "-shared", obj, "-L", PKG, "-l:libapbv.so", "-Wl,-rpath,$ORIGIN", "-L", torch_lib, "-ltorch_python", "-ltorch_cpu", "-lc10",
             "-o", MARSHAL])


def build(verbose: bool = True, extra=()) -> str:
    os.makedirs(OBJ, exist_ok=True)
    marshal = marshal_commands()

    def compile_one(item):
        src, own = item
        obj = os.path.join(OBJ, src.replace(".hip", ".o"))
        cmd = [HIPCC, *FLAGS, *own, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        return obj

    with ThreadPoolExecutor(max_workers=min(len(SOURCES) + 1, 8)) as pool:
        marshal_obj = pool.submit(subprocess.run, marshal[0], check=True) if marshal else None
        objs = list(pool.map(compile_one, SOURCES.items()))
        if marshal_obj:
            marshal_obj.result()
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    if marshal:
        subprocess.run(marshal[1], check=True)
    return LIB


if __name__ == "__main__":
    build(extra=sys.argv[1:])
