"""Build libmosaic.so in-tree with hipcc for gfx950.

Every HIP source under csrc/ is compiled to an object file under _build/ and
linked into paper_2607_29221_amd/libmosaic.so; csrc/binding.cpp, the Python
binding's native marshalling, is compiled (host code only, against torch's
headers) into paper_2607_29221_amd/_binding.so. Run ``python -m
paper_2607_29221_amd.build`` (or ``__graft_entry__.build()``). Beside the
library the build writes libmosaic.so.sources, a digest of every file it was
built from (csrc/, include/) and of the compiler flags, and beside the binding
_binding.so.sources, which adds the torch and Python it was compiled against;
the loader refuses a
library whose digest no longer matches the sources.
"""
from __future__ import annotations

import hashlib
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(HERE, "libmosaic.so")
BINDING = os.path.join(HERE, "_binding.so")
STAMP = LIB + ".sources"
BINDING_STAMP = BINDING + ".sources"
INCLUDE = os.path.join(ROOT, "include")
ARCH = os.environ.get("MOSAIC_OFFLOAD_ARCH", "gfx950")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCES = ["abi.cpp", "elementwise.hip", "ring_gemm.hip", "ring_gemm_skinny.hip", "ring_gemv.hip", "hadamard.hip", "quantize.hip",
           "sparse.hip", "sparse_terms.hip", "abi_terms.cpp", "secure_input.hip", "hadamard28.hip", "probe.hip"]
FLAGS = [f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-x", "hip",
         # keep the compiler from forming packed fp32 instructions
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-command-line-argument"]


def source_digest() -> str:
    """sha256 over the names and contents of every file under csrc/ and
    include/, the compiler flags and the target architecture."""
    h = hashlib.sha256()
    h.update(" ".join(FLAGS + [HIPCC]).encode())
    for d in (CSRC, INCLUDE):
        for name in sorted(os.listdir(d)):
            path = os.path.join(d, name)
            if os.path.isfile(path):
                h.update(name.encode() + b"\0")
                with open(path, "rb") as f:
                    h.update(f.read())
    return h.hexdigest()


# hipcc's clang as a plain C++ compiler, without the HIP runtime: the binding
# reaches the library through the addresses it is given.
BINDING_FLAGS = ["-x", "c++", "-no-hip-rt", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall"]


def binding_digest() -> str:
    """sha256 over the binding's sources and flags and the torch and Python
    whose headers, layouts and interfaces are compiled into it."""
    import torch
    h = hashlib.sha256()
    h.update(" ".join(BINDING_FLAGS + [HIPCC, torch.__version__, str(torch._C._GLIBCXX_USE_CXX11_ABI),
                                       sysconfig.get_config_var("SOABI") or sys.version]).encode())
    for path in (os.path.join(CSRC, "binding.cpp"), os.path.join(CSRC, "dispatch.h"),
                 os.path.join(INCLUDE, "mosaic.h")):
        with open(path, "rb") as f:
            h.update(f.read())
    return h.hexdigest()


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{res.stdout}\n{res.stderr}")
    return obj


def _build_binding() -> None:
    import torch
    root = os.path.dirname(torch.__file__)
    digest = binding_digest()
    tmp = BINDING + ".tmp"
    cmd = [HIPCC] + BINDING_FLAGS + [
        f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
        f"-I{root}/include", f"-I{root}/include/torch/csrc/api/include", f"-I{sysconfig.get_paths()['include']}",
        os.path.join(CSRC, "binding.cpp"), "-o", tmp, f"-L{root}/lib", "-ltorch_python", "-ltorch_cpu", "-lc10"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"compiling the binding failed:\n{res.stdout}\n{res.stderr}")
    os.replace(tmp, BINDING)
    with open(BINDING_STAMP, "w") as f:
        f.write(digest + "\n")


def build(verbose: bool = False) -> str:
    digest = source_digest()
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 1)) as ex:
        binding = ex.submit(_build_binding)
        objs = list(ex.map(_compile, SOURCES))
        binding.result()
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp] + objs
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed:\n{res.stdout}\n{res.stderr}")
    os.replace(tmp, LIB)
    with open(STAMP, "w") as f:
        f.write(digest + "\n")
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
