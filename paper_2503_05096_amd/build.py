"""Builds libadaspec.so (the C-ABI library) from csrc/*.hip (device + host code) and csrc/*.cpp
(host-only code) for gfx950 with hipcc, and _fastcall.so (the Python binding's native call path) with g++."""
from __future__ import annotations

import glob
import hashlib
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
BUILD_DIR = os.path.join(HERE, "_build")
LIB_PATH = os.path.join(HERE, "libadaspec.so")
FASTCALL_SOURCE = os.path.join(HERE, "csrc_python", "fastcall.cpp")
FASTCALL_PATH = os.path.join(HERE, "_fastcall.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
    # packed-FP32 instructions stay off (scalar fp32 code only)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def build_fastcall(verbose: bool = False, out: str = FASTCALL_PATH, defines=()) -> str:
    """The extension module uses torch's and Python's headers only (no HIP), so the host compiler builds it."""
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I", os.path.join(root, "include"), "-I", os.path.join(root, "include", "torch", "csrc", "api", "include"),
           "-I", sysconfig.get_paths()["include"], f'-DADASPEC_TORCH_VERSION="{torch.__version__}"',
           *(f"-D{d}" for d in defines), FASTCALL_SOURCE, "-o", out,
           "-L", os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed on {FASTCALL_SOURCE}:\n{r.stderr}")
    return out


def _sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.cpp")))


def _object(src: str, tag: str = "") -> str:
    return os.path.join(BUILD_DIR, os.path.basename(src).replace(".", "_") + tag + ".o")


def _compile(src: str, obj: str, defines=(), verbose: bool = False) -> str:
    cmd = [HIPCC, *FLAGS, *(f"-D{d}" for d in defines), "-I", INCLUDE, "-c", src, "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr}")
    return r.stderr


def _link(objects, out: str) -> str:
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", out, *objects], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    return out


def _inputs():
    return sorted(glob.glob(os.path.join(CSRC, "*")) + glob.glob(os.path.join(INCLUDE, "*")))


def source_key(defines=()) -> str:
    """What the library is made from: a digest of its sources, headers, flags and `defines`."""
    h = hashlib.sha256(repr((FLAGS, tuple(defines))).encode())
    for path in _inputs():
        h.update(os.path.basename(path).encode() + b"\0" + open(path, "rb").read())
    return h.hexdigest()[:16]


def _includes(path: str, header: str) -> bool:
    """Whether the file includes csrc/`header`, also through other headers of csrc."""
    names = re.findall(r'#include "([^"]+)"', open(path).read())
    return header in names or any(_includes(os.path.join(CSRC, n), header) for n in names if os.path.exists(os.path.join(CSRC, n)))


def build_variant(out: str, tag: str, defines, header: str, jobs: int = 8) -> str:
    """The library with `defines` for the sources that include `header`. The other objects are the library's own where
    they are there and newer than every source."""
    newest = max(os.path.getmtime(p) for p in _inputs())
    os.makedirs(BUILD_DIR, exist_ok=True)

    def obj(src):
        own = _object(src)
        if _includes(src, header):
            own = _object(src, "_" + tag)
            _compile(src, own, defines)
        elif not os.path.exists(own) or os.path.getmtime(own) < newest:
            own = _object(src, "_" + tag)
            _compile(src, own)
        return own
    with ThreadPoolExecutor(jobs) as ex:
        return _link(list(ex.map(obj, _sources())), out)


def build_library(verbose: bool = False, jobs: int = 8) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    sources = _sources()
    objects = [_object(s) for s in sources]

    with ThreadPoolExecutor(jobs) as ex:
        fastcall = ex.submit(build_fastcall, verbose)
        logs = list(ex.map(lambda s: _compile(s, _object(s), verbose=verbose), sources))
    try:
        fastcall.result()
    except Exception as e:      # no host compiler, no Python headers: the binding makes its calls in Python then
        if os.path.exists(FASTCALL_PATH):
            os.remove(FASTCALL_PATH)                # never one that is older than the library
        print(f"_fastcall.so was not built, calls from Python take some microseconds longer: {e}", file=sys.stderr)
    if verbose:
        for log in logs:
            # hipcc's host pass does not know the device-only feature flag: harmless
            keep = [l for l in log.splitlines() if "packed-fp32-ops" not in l and l.strip()]
            if keep:
                print("\n".join(keep))
    return _link(objects, LIB_PATH)


if __name__ == "__main__":
    print(build_library(verbose="-v" in sys.argv))
