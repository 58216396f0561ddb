"""Builds libbiq.so (the HIP kernels and their C ABI) for gfx950 with hipcc, and the extension module _calls (the calls
from Python into it, host code; needs g++ and this interpreter's headers), in-tree.

One translation unit per kernel family (csrc/*.hip), compiled side by side and linked into one
shared library; objects go to paper_2005_09904_amd/_build/ (not tracked)."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
OBJ_DIR = os.path.join(PKG_DIR, "_build")
LIB_PATH = os.path.join(PKG_DIR, "libbiq.so")
# (named for the interpreter it is built for: another one finds none, rather than one with other object layouts)
CALLS_PATH = os.path.join(PKG_DIR, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))
CALLS_SOURCE = os.path.join(CSRC, "py_calls.cpp")
SOURCES = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
HEADERS = sorted(glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.inc"))) + [
    os.path.join(ROOT, "include", "biq.h")]

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    # packed fp32 VALU forms are kept out of the generated code on purpose
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def is_stale() -> bool:
    if not os.path.exists(LIB_PATH) or not os.path.exists(CALLS_PATH):
        return True
    built = min(os.path.getmtime(LIB_PATH), os.path.getmtime(CALLS_PATH))
    return any(os.path.getmtime(p) > built for p in SOURCES + HEADERS + [CALLS_SOURCE])


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass warns that it does not know the packed-fp32 feature; that is expected
    out = "\n".join(l for l in proc.stdout.splitlines() if "packed-fp32-ops" not in l)
    if proc.returncode != 0:
        raise RuntimeError("%s failed: %s\n%s" % (cmd[0], " ".join(cmd), out))
    if verbose and out.strip():
        print(out)


def build_library(verbose: bool = False, jobs: int | None = None) -> str:
    """Compiles every HIP source and links libbiq.so (always recompiles). Returns the library path."""
    hipcc = os.environ.get("HIPCC", "hipcc")
    os.makedirs(OBJ_DIR, exist_ok=True)
    inc = ["-I" + os.path.join(ROOT, "include"), "-I" + CSRC]
    tag = ".%d" % os.getpid()
    objs = [os.path.join(OBJ_DIR, os.path.basename(s)[:-4] + tag + ".o") for s in SOURCES]
    jobs = jobs or min(len(SOURCES), int(os.environ.get("MAX_JOBS", "0")) or os.cpu_count() or 1, 16)
    try:
        with ThreadPoolExecutor(max_workers=jobs) as pool:
            list(pool.map(lambda so: _run([hipcc] + HIPCC_FLAGS + inc + ["-c", so[0], "-o", so[1]], verbose),
                          zip(SOURCES, objs)))
        tmp = LIB_PATH + ".tmp" + tag
        _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", tmp], verbose)
        os.replace(tmp, LIB_PATH)
        tmp = CALLS_PATH + ".tmp" + tag
        _run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
              inc[0], "-I" + sysconfig.get_paths()["include"], CALLS_SOURCE, "-o", tmp], verbose)
        os.replace(tmp, CALLS_PATH)
    finally:
        for o in objs:
            if os.path.exists(o):
                os.remove(o)
    return LIB_PATH


if __name__ == "__main__":
    print(build_library(verbose=True))
    sys.exit(0)
