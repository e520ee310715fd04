"""Builds libcts.so (the HIP kernels and the C ABI) in-tree for gfx950, and
_marshal.so (the Python binding's tensor checks, host code).

    python -m paper_2407_00066_amd.build

Every translation unit is compiled with hipcc for gfx950 only, with the
packed-fp32 instructions disabled, then linked into one shared library next
to this file.  The public header is include/cts.h at the repository root.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libcts.so")
MARSHAL = os.path.join(PKG, "_marshal.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

FLAGS = ["--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC", "-Wall",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", INCLUDE, "-I", CSRC]


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


# host code under AddressSanitizer and UndefinedBehaviorSanitizer (the
# device code is compiled as always): the sanitizer check of the CPU tests
SAN_FLAGS = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
             "-Xarch_host", "-fno-sanitize-recover=undefined", "-Xarch_host", "-fno-omit-frame-pointer",
             "-Xarch_host", "-g"]


def _compile(src: str, build_dir: str = BUILD, sanitize: bool = False) -> str:
    obj = os.path.join(build_dir, os.path.basename(src) + ".o")
    cmd = [HIPCC] + FLAGS + (SAN_FLAGS if sanitize else []) + ["-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed on %s:\n%s%s" % (src, r.stdout, r.stderr))
    noise = "'-packed-fp32-ops' is not a recognized feature"
    msgs = [ln for ln in (r.stdout + r.stderr).splitlines() if ln.strip() and noise not in ln]
    if msgs:
        print("\n".join(msgs), file=sys.stderr)
    return obj


def build_marshal() -> str:
    """Compile the binding's tensor checks (csrc/marshal.cpp: host code, torch's
    C++ API) into _marshal.so."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension

    tmp = MARSHAL + ".tmp%d" % os.getpid()
    inc = [a for d in cpp_extension.include_paths() + [sysconfig.get_paths()["include"]] for a in ("-isystem", d)]
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           '-DCTS_TORCH_VERSION="%s"' % torch.__version__] + inc + \
          [os.path.join(CSRC, "marshal.cpp"), "-o", tmp, "-L" + lib, "-ltorch_python", "-ltorch_cpu", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed on marshal.cpp:\n%s%s" % (r.stdout, r.stderr))
    os.replace(tmp, MARSHAL)
    return MARSHAL


def build(verbose: bool = True, out: str | None = None, sanitize: bool = False) -> str:
    """Compile every source and link libcts.so (into `out` if given; with
    sanitize, the host code under AddressSanitizer and
    UndefinedBehaviorSanitizer, linked to the shared sanitizer runtime)."""
    lib = out or LIB
    build_dir = os.path.join(os.path.dirname(lib), "_build_san") if sanitize else BUILD
    os.makedirs(build_dir, exist_ok=True)
    srcs = sources()
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs) + 1)) as ex:
        marshal = ex.submit(build_marshal) if out is None else None
        objs = list(ex.map(lambda s_: _compile(s_, build_dir, sanitize), srcs))
    tmp = lib + ".tmp%d" % os.getpid()
    cmd = [HIPCC, "--offload-arch=" + ARCH, "-shared", "-fPIC", "-o", tmp] + objs
    if sanitize:
        cmd += ["-fsanitize=address,undefined", "-shared-libsan"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s%s" % (r.stdout, r.stderr))
    os.replace(tmp, lib)
    if marshal is not None:
        marshal.result()
    if verbose:
        print("built", lib)
    return lib


if __name__ == "__main__":
    build()
