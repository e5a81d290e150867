"""Builds libcascade_attn.so (gfx950) in-tree with hipcc, and the Python extension beside it.  Used by __graft_entry__.build()."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.environ.get("CASCADE_ATTN_LIB") or os.path.join(PKG, "libcascade_attn.so")

SOURCES = ["ca_meta.cpp", "ca_api.cpp", "ca_sched.cpp", "rope_cache.hip", "attn_f32.hip", "attn_bf16.hip", "mfma_peak.hip", "gemm_bf16.hip", "gemm_rows.hip", "gemm_tiles.hip"]

# packed fp32 instructions are kept off for all device code
DEVICE_FLAGS = ["-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
# Loops begin at a multiple of 64 bytes there: where the loop of the 128 x 128 tile began 28 bytes behind one (a change of its
# arguments had moved it from 16), the same instructions took 3 % longer: 3011 x 1096 x 4864 37.7 us, 36.5 now, 15272 x 208 x
# 4224 34.7 / 33.6, 3146 x 1064 x 3456 28.2 / 27.2.
FILE_FLAGS = {"gemm_tiles.hip": ["-falign-loops=64"]}


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found")
    return exe


def calls_path() -> str:
    """The Python extension (csrc/py_calls.cpp) fits one Python and one torch, which its name says."""
    import torch
    return os.path.join(PKG, f"_calls.{sys.implementation.cache_tag}.torch-{torch.__version__}.so")


def calls_command(out: str) -> list:
    """The extension holds no device code: g++ against the headers of torch and of HIP's host side."""
    import torch
    torch = torch.__path__[0]
    return [shutil.which("g++") or "g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            "-I", os.path.join(ROOT, "include"), "-I", os.path.join(torch, "include"),
            "-I", os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), "-I", sysconfig.get_paths()["include"],
            os.path.join(CSRC, "py_calls.cpp"), "-L", os.path.join(torch, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python",
            "-o", out]


def _finish(src: str, p: subprocess.Popen, verbose: bool = False) -> None:
    out, _ = p.communicate()
    if p.returncode != 0:
        raise RuntimeError(f"the compiler failed on {src}:\n{out}")
    if verbose and out.strip():
        print(out)


def build_calls(beside=None) -> None:
    """The Python extension, while `beside` runs if it is given; the file takes its place when it is whole."""
    path = calls_path()
    part = f"{path}.{os.getpid()}.part"
    p = subprocess.Popen(calls_command(part), stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    try:
        if beside:
            beside()
        _finish("py_calls.cpp", p)
        os.replace(part, path)
    finally:
        if p.returncode is None:
            p.communicate()
        if os.path.exists(part):
            os.remove(part)


def build_library(verbose: bool = False, extra=(), bdir: str | None = None) -> None:
    objs = []
    bdir = bdir or os.path.join(PKG, "_build")
    os.makedirs(bdir, exist_ok=True)
    # the hand-scheduled main loops are emitted as inline-assembly includes
    for core in ("attn_core", "attn_core16", "gemm_core", "gemm_rows"):
        subprocess.run([sys.executable, os.path.join(CSRC, f"gen_{core}.py"), os.path.join(bdir, f"{core}_gfx950.inc")],
                       check=True, stdout=None if verbose else subprocess.DEVNULL)
    common = ["-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "-I", os.path.join(ROOT, "include"),
              "-I", CSRC, "-I", bdir, "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option"] + DEVICE_FLAGS + list(extra)
    procs = []
    for src in SOURCES:
        obj = os.path.join(bdir, src + ".o")
        cmd = [hipcc(), "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj] + common + FILE_FLAGS.get(src, [])
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    for src, p in procs:
        _finish(src, p, verbose)
    cmd = [hipcc(), "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB] + objs
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout)


def build(verbose: bool = False, extra=(), bdir: str | None = None) -> str:
    build_calls(beside=lambda: build_library(verbose, extra, bdir))
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
