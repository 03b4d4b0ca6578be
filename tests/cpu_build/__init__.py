"""The library compiled for the CPU (its kernels on fibers) for tests that need no
GPU: build() compiles it for a few species counts, use() points the Python
binding at it, with CPU tensors in the place of device tensors."""
import ctypes as C
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest
import torch

from paper_2202_02319_amd import _lib, htr

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
CSRC = os.path.join(ROOT, "paper_2202_02319_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"


def build(out, species):
    if not os.path.exists(CLANG):
        pytest.skip(f"{CLANG} is missing")
    out = str(out)
    objs = []
    for f in os.listdir(CSRC):
        with open(os.path.join(CSRC, f)) as fh:
            s = fh.read()
        # an alignment before the storage class, which __shared__ and __device__ become
        s = re.sub(r"__shared__ (alignas\(\d+\))", r"\1 __shared__", s)
        if f == "htr_dev.h":
            cases = " ".join(f"case {n}: return CALL({n});" for n in species)
            s = re.sub(r"#define HTR_NS_SWITCH\(ns, CALL\)(.*\\\n)+.*\}",
                       f"#define HTR_NS_SWITCH(ns, CALL) switch (ns) {{ {cases} default: return hipErrorInvalidValue; }}",
                       s)
        with open(os.path.join(out, f), "w") as fh:
            fh.write(s)
        if not f.endswith(".h"):
            objs.append(os.path.join(out, f))
    objs.append(os.path.join(HERE, "run.cpp"))

    def compile_(src):
        obj = os.path.join(out, os.path.basename(src) + ".o")
        subprocess.run([CLANG, "-std=c++17", "-O1", "-fPIC", "-w", "-mfma", "-ffp-contract=fast-honor-pragmas", "-x", "c++",
                        *(["-DCPU_COUNT_CALLS"] if src.endswith(".hip") else []), "-I", HERE, "-I", os.path.join(ROOT, "include"), "-I", out, "-c", src, "-o", obj], check=True)
        return obj
    with ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(compile_, objs))
    lib = os.path.join(out, "libhtr_cpu.so")
    subprocess.run([CLANG, "-shared", *objs, "-o", lib], check=True)
    return lib


def _ptr(t):
    if t is None:
        return None
    assert t.dtype in (torch.float64, torch.uint8) and t.is_contiguous()
    return C.c_void_p(t.data_ptr())


def use(lib, mp):
    """The binding on lib until mp (a MonkeyPatch) is undone."""
    mp.setattr(_lib, "LIB_PATH", lib)
    mp.setattr(_lib, "_lib", None)
    mp.setattr(htr, "_ptr", _ptr)
    mp.setattr(htr, "_stream", lambda stream: None)
    L = _lib.load()
    L.cpu_capture_end.restype = C.c_void_p
    L.cpu_replay.argtypes = [C.c_void_p]
    L.cpu_calls.restype = C.c_longlong
    return L
