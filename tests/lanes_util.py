"""csrc/lanes.h (the rules by which kernels deal out their lanes) compiled for the CPU."""
import ctypes
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2102_02989_amd", "csrc")


def build(directory, source):
    if not shutil.which("g++") or not os.path.isdir("/opt/rocm/include/hip"):
        pytest.skip("g++ and the HIP headers are needed")
    src, lib = os.path.join(str(directory), "l.cpp"), os.path.join(str(directory), "l.so")
    with open(src, "w") as fh:
        fh.write(source)
    cmd = ["g++", "-std=c++17", "-O2", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC,
           "-D__align__(n)=__attribute__((aligned(n)))", "-o", lib, src]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return ctypes.CDLL(lib)
