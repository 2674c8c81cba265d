"""Builds host_checks.cpp against the library and loads it."""
import ctypes
import functools
import os
import subprocess
import tempfile

from paper_2411_18906_amd import build_lib

HERE = os.path.dirname(os.path.abspath(__file__))


@functools.lru_cache(maxsize=None)
def lib():
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    out = os.path.join(tempfile.mkdtemp(prefix="pyhea_host_"), "host_checks.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-w",
                    "-I", os.path.join(rocm, "include"), "-I", os.path.join(build_lib.ROOT, "include"),
                    "-I", build_lib.CSRC, os.path.join(HERE, "host_checks.cpp"), build_lib.LIB,
                    "-Wl,-rpath," + os.path.dirname(build_lib.LIB), "-o", out], check=True)
    return ctypes.CDLL(out)
