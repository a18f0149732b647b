"""The library's host/device functions (index and hash rules of csrc/tang_internal.hpp) as a
small host library of their own, for tests that need no GPU."""
import ctypes
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2601_03187_amd", "csrc")


def compile_host(directory, body: str) -> ctypes.CDLL:
    """`body` (C++ in namespace tang, its entries extern "C") with the internal header before it."""
    src, out = os.path.join(directory, "internal.cpp"), os.path.join(directory, "internal.so")
    with open(src, "w") as f:
        f.write('#include "tang_internal.hpp"\nusing namespace tang;\n' + body)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O2", "-w", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(rocm, "include"), "-I", CSRC, "-o", out, src], check=True)
    return ctypes.CDLL(out)
