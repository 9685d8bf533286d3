"""Builds libvtrace.so in-tree with hipcc for gfx950.

``python -m paper_1802_01561_amd.build`` compiles every ``csrc/*.hip`` file
to an object in parallel and links the shared library next to this file, and
compiles ``csrc/fast_call.cpp`` (the torch binding's argument marshalling, host
code only) to ``_fast_call.so`` beside it.
"""

from __future__ import annotations

import concurrent.futures
import os
import shutil
import subprocess
import sys
import sysconfig

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
REPO_DIR = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
BUILD_DIR = os.path.join(PKG_DIR, "_build")
LIB_PATH = os.path.join(PKG_DIR, "libvtrace.so")
FAST_CALL_PATH = os.path.join(PKG_DIR, "_fast_call.so")
ARCH = "gfx950"

# -packed-fp32-ops: keep hipcc from forming packed fp32 ALU instructions.
HIP_FLAGS = [
    f"--offload-arch={ARCH}",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-Wall",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(REPO_DIR, "include"),
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: install ROCm or set HIPCC")


def _compile(src: str, extra: list[str], build_dir: str) -> str:
    obj = os.path.join(build_dir, os.path.basename(src) + ".o")
    cmd = [hipcc(), *HIP_FLAGS, *extra, "-c", src, "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{' '.join(cmd)}\n{res.stdout}\n{res.stderr}")
    return obj


def build(extra_flags: list[str] | None = None, verbose: bool = False, *, lib_path: str = LIB_PATH,
          build_dir: str = BUILD_DIR, link_flags: list[str] | None = None) -> str:
    """Compiles and links libvtrace.so (or, with lib_path and build_dir, a
    variant of it such as the host-instrumented one); returns its path."""
    extra = list(extra_flags or [])
    os.makedirs(build_dir, exist_ok=True)
    srcs = sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(lambda s: _compile(s, extra, build_dir), srcs))
    tmp = lib_path + ".tmp"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", *(link_flags or []), "-o", tmp, *objs]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed:\n{' '.join(cmd)}\n{res.stdout}\n{res.stderr}")
    os.replace(tmp, lib_path)
    if verbose:
        print(f"built {lib_path}")
    return lib_path


def build_fast_call(verbose: bool = False) -> str:
    """Compiles _fast_call.so against the installed torch; returns its path."""
    import torch
    from torch.utils import cpp_extension

    tmp = FAST_CALL_PATH + ".tmp"
    libs = cpp_extension.library_paths()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I", os.path.join(REPO_DIR, "include"), "-I", sysconfig.get_paths()["include"],
           *(f"-I{p}" for p in cpp_extension.include_paths()), os.path.join(CSRC, "fast_call.cpp"), "-o", tmp,
           *(f"-L{p}" for p in libs), "-ltorch_python", "-ltorch_cpu", "-lc10", *(f"-Wl,-rpath,{p}" for p in libs)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"compilation failed:\n{' '.join(cmd)}\n{res.stdout}\n{res.stderr}")
    os.replace(tmp, FAST_CALL_PATH)
    if verbose:
        print(f"built {FAST_CALL_PATH}")
    return FAST_CALL_PATH


if __name__ == "__main__":
    build_fast_call(verbose=True)
    build(sys.argv[1:], verbose=True)
