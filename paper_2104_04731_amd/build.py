"""Compile the HIP library for gfx950 in-tree (hipcc cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libconv2d_int8.so")
SOURCES = ["api.cpp", "selector.cpp", "igemm_mfma.hip", "band_mfma.hip", "resident_mfma.hip", "stream_mfma.hip", "layout_kernels.hip", "window_mfma.hip", "stencil_mfma.hip",
           "panel_mfma.hip", "pointwise_mfma.hip"]
HEADERS = [os.path.join(CSRC, "kernels.h"), os.path.join(CSRC, "rewrite_bodies.h"), os.path.join(CSRC, "act_requant.h"), os.path.join(CSRC, "act_store.h"), os.path.join(CSRC, "desc_check.h"), os.path.join(CSRC, "launch.h"), os.path.join(CSRC, "store_past.h"), os.path.join(CSRC, "panel_fill.h"), os.path.join(CSRC, "window_fill.h"), os.path.join(CSRC, "window_walk.h"),
           os.path.join(os.path.dirname(PKG), "include", "conv2d_int8.h")]

NATIVE_SOURCE = "py_native.cpp"                    # the Python side of the tensor-taking calls: host code, no kernels
NATIVE = os.path.join(PKG, "_native.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
    "-Wno-unused-command-line-argument",
    # keep the compiler from forming packed-fp32 ALU ops (harmless host-side warning)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def stale() -> bool:
    if not (os.path.exists(LIB) and os.path.exists(NATIVE)):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(NATIVE))
    deps = [os.path.join(CSRC, s) for s in [*SOURCES, NATIVE_SOURCE]] + HEADERS
    return any(os.path.getmtime(d) > t for d in deps)


def native_commands():
    """Compile and link lines of the extension module: torch's headers and libraries (it is handed the loaded library)."""
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    obj = os.path.join(CSRC, "py_native.o")
    compile_cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
                   f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
                   "-isystem", os.path.join(root, "include"), "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"),
                   "-isystem", "/opt/rocm/include", "-isystem", sysconfig.get_paths()["include"],
                   "-c", os.path.join(CSRC, NATIVE_SOURCE), "-o", obj]
    link_cmd = ["g++", "-shared", "-fPIC", "-o", NATIVE, obj, "-ldl",
                "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-ltorch_hip", "-lc10", "-lc10_hip"]
    return compile_cmd, link_cmd


def build_library(verbose: bool = False) -> str:
    from concurrent.futures import ThreadPoolExecutor

    def compile_one(s):
        src = os.path.join(CSRC, s)
        obj = os.path.join(CSRC, os.path.splitext(s)[0] + ".o")
        cmd = ["hipcc", *HIPCC_FLAGS, "-x", "hip", "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        return obj

    # the translation units are independent: compile them side by side (the GEMM kernel's file dominates)
    native_compile, native_link = native_commands()
    with ThreadPoolExecutor(max_workers=min(len(SOURCES) + 1, os.cpu_count() or 1, 8)) as pool:
        native = pool.submit(subprocess.check_call, native_compile)
        objs = list(pool.map(compile_one, SOURCES))
        native.result()
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    if verbose:
        print(" ".join(native_link), flush=True)
    subprocess.check_call(native_link)
    return LIB


if __name__ == "__main__":
    build_library(verbose=True)
    print(LIB)
    sys.exit(0)
