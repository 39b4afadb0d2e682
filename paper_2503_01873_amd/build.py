"""Builds libpasa.so (hipcc, gfx950) and the binding's extension _calls (C) in-tree.  `python -m paper_2503_01873_amd.build`."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libpasa.so")
CALLS = os.path.join(PKG, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))      # for this interpreter: others do not load it
SOURCES = ["pasa_api.hip", "pasa_kernels.hip", "pasa_fwd4.hip", "pasa_rows.hip", "pasa_shift_gemm.hip"]

FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    "-ffp-contract=off",          # every rounding the method states is a separate operation
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-mllvm", "-amdgpu-kernarg-preload-count=16",   # a kernel's first arguments come in registers: a row of 32768 keys 16.05 -> 15.8 us
    "-Wall",
    "-Wno-unused-function",
]


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found; libpasa cannot be built")
    return exe


def build_calls(verbose: bool = False) -> str | None:
    """None, with a note, where Python's headers are not installed: the binding does without (through ctypes)."""
    include = sysconfig.get_paths()["include"]
    if not os.path.exists(os.path.join(include, "Python.h")):
        print(f"no Python.h in {include}: the binding's calls stay with ctypes, 3 us slower each", file=sys.stderr, flush=True)
        return None
    cmd = [shutil.which("gcc") or hipcc(), "-O2", "-std=c11", "-fPIC", "-shared", "-Wall", "-I", include,
           "-I", os.path.join(ROOT, "include"), os.path.join(CSRC, "calls.c"), "-o", CALLS]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("the binding's extension does not compile:\n" + res.stdout + res.stderr)
    return CALLS


def build(verbose: bool = False, extra_flags=(), out: str = LIB) -> str:
    cmd = [hipcc(), *FLAGS, *extra_flags, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           *[os.path.join(CSRC, s) for s in SOURCES], "-o", out]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    log = (res.stdout + res.stderr)
    # hipcc's host pass does not know the packed-fp32 feature name; that warning is expected
    shown = "\n".join(l for l in log.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + log)
    if verbose and shown.strip():
        print(shown)
    build_calls(verbose)
    return out


if __name__ == "__main__":
    print(build(verbose=True, extra_flags=sys.argv[1:]))
