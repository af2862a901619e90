"""Build libdpclip.so (HIP, gfx950 only) in-tree with hipcc, and the Python extension over it with g++."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG_DIR, "csrc")
INCLUDE = os.path.join(os.path.dirname(PKG_DIR), "include")
LIB_PATH = os.path.join(PKG_DIR, "libdpclip.so")
NATIVE_PATH = os.path.join(PKG_DIR, "_native.so")
BUILD_DIR = os.path.join(PKG_DIR, "_build")

SOURCES = ["dp_api.hip", "dp_update.hip", "dp_rowwise.hip", "dp_gram.hip", "dp_wgemm.hip", "dp_tied.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-I" + INCLUDE, "-I" + CSRC,
    # the compiler must not form packed-fp32 instructions on its own
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-result",
]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    return "hipcc"


def _compile(src: str) -> str:
    obj = os.path.join(BUILD_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc()] + HIPCC_FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr}")
    return obj


def _run(cmd, what):
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{what} failed:\n{r.stderr}")


def _compile_native() -> str:
    import torch

    obj, top = os.path.join(BUILD_DIR, "native.o"), os.path.dirname(torch.__file__)
    includes = [INCLUDE, os.path.join(top, "include"), os.path.join(top, "include", "torch", "csrc", "api", "include"),
                sysconfig.get_paths()["include"]]
    _run(["g++", "-O2", "-std=c++17", "-fPIC", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
         + ["-I" + i for i in includes] + ["-c", os.path.join(CSRC, "native.cpp"), "-o", obj], "g++ on native.cpp")
    return obj


def _link_native(obj, lib, out):
    """Finds libdpclip.so (here `lib`, which bears that name inside) beside itself; libtorch is in the process before it is imported."""
    import torch

    top = os.path.join(os.path.dirname(torch.__file__), "lib")
    _run(["g++", "-shared", "-o", out, obj, lib, "-Wl,-rpath,$ORIGIN", "-L" + top, "-ltorch_python", "-ltorch_cpu", "-lc10"],
         "link of _native.so")


def build_library(verbose: bool = False) -> str:
    """Compile every source and link the shared library and the extension; always rebuilds.  Neither file is replaced before both are
    linked: the extension has the library's argument lists compiled in."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(len(SOURCES) + 1, os.cpu_count() or 1)) as ex:
        native = ex.submit(_compile_native)
        objs = list(ex.map(_compile, SOURCES))
        native = native.result()
    lib, ext = LIB_PATH + ".tmp", NATIVE_PATH + ".tmp"
    # (the name that whoever links against it finds it by, whatever the file is called while it is written)
    _run([_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-Wl,-soname,libdpclip.so", "-o", lib] + objs, "link")
    _link_native(native, lib, ext)
    os.replace(lib, LIB_PATH)
    os.replace(ext, NATIVE_PATH)
    if verbose:
        print("built", LIB_PATH, "and", NATIVE_PATH, file=sys.stderr)
    return LIB_PATH


if __name__ == "__main__":
    build_library(verbose=True)
