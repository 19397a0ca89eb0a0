"""Build librsgdf.so for gfx950 with hipcc (in-tree, no JIT cache)."""
from __future__ import annotations

import concurrent.futures
import glob
import hashlib
import os
import shutil
import subprocess
import sys

try:
    from . import asm_check
except ImportError:  # run as a script
    import asm_check

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "librsgdf.so")
SOURCES = ["sr3c.hip", "fold.hip", "lr.hip", "learned.hip", "j2c.hip", "df.hip", "coulomb.hip", "capi.cpp"]
ARCH = os.environ.get("RSGDF_ARCH", "gfx950")


def source_hash() -> str:
    """SHA-256 (first 16 hex digits) over the library's sources: every file of
    csrc/ and the public headers, by name and content.  The build bakes it into
    the library (rsgdf_source_hash) and the binding compares it on load."""
    h = hashlib.sha256()
    inc = os.path.join(ROOT, "include")
    for d in (CSRC, inc):
        for f in sorted(os.listdir(d)):
            if f.endswith((".hip", ".cpp", ".h")):
                h.update(f.encode() + b"\0")
                with open(os.path.join(d, f), "rb") as fh:
                    h.update(fh.read())
    return h.hexdigest()[:16]


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found")


def flags():
    return ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-I", os.path.join(ROOT, "include"),
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-munsafe-fp-atomics",
            "-Wno-unused-command-line-argument"]


def check_assembly(path: str) -> int:
    """Refuse device code in which a per-lane instruction precedes an exec restore
    (asm_check), or whose text the check no longer understands."""
    with open(path) as fh:
        restores, found = asm_check.check(fh.read())
    if found:
        raise RuntimeError(f"{path}: per-lane instructions in front of an exec restore, where the lanes that left a "
                           "divergent region lose the value (fewer live registers in the kernel, or another "
                           "compiler):\n" + "\n".join(f"  {f}, line {n}: {i}" for f, n, i in found))
    if restores == 0:
        raise RuntimeError(f"{path}: no exec restore found; the check of the assembly does not read it")
    return restores


def _compile(src: str, defs=()) -> str:
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    tmp = os.path.join(BUILD, "tmp_" + src.replace(".", "_"))
    shutil.rmtree(tmp, ignore_errors=True)
    os.makedirs(tmp)
    # the device code is assembled from the text that -save-temps leaves (capi.cpp has
    # none, and its host code is not put through a text)
    kernels = src.endswith(".hip")
    tobj = os.path.join(tmp, os.path.basename(obj))
    cmd = [hipcc(), *flags(), *defs, *(["-save-temps=obj"] if kernels else []), "-x", "hip", "-c",
           os.path.join(CSRC, src), "-o", tobj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    if kernels:
        asm = glob.glob(os.path.join(tmp, f"*-hip-amdgcn-amd-amdhsa-{ARCH}*.s"))
        if len(asm) != 1:
            raise RuntimeError(f"{src}: expected one device assembly text under {tmp}, found {len(asm)}")
        check_assembly(asm[0])
    os.replace(tobj, obj)
    shutil.rmtree(tmp)
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    defs = [f'-DRSGDF_SOURCE_HASH="{source_hash()}"']
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(lambda src: _compile(src, defs), SOURCES))
    tmp = LIB + ".tmp"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs, "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
