"""The library's selection, gather and decode kernels compiled for the host CPU (see hip/hip_runtime.h), behind the same C ABI with
host pointers. Array indexes are checked (a bad one traps), and memory that the kernels may not touch can be given without access."""
import ctypes
import mmap
import os
import pathlib
import shutil
import subprocess

import numpy as np

from paper_2602_08686_amd import binding as B

HERE = pathlib.Path(__file__).resolve().parent
ROOT = HERE.parents[1]
CXX = next((c for c in ("/opt/rocm/llvm/bin/clang++", shutil.which("clang++")) if c and os.path.exists(c)), None)
HOOK = ctypes.CFUNCTYPE(None, ctypes.c_int, ctypes.c_int)


def build(where) -> str:
    """Compile into the folder `where`; returns the library's path."""
    objs, procs = [], []
    csrc = ROOT / "paper_2602_08686_amd" / "csrc"
    for src in (csrc / "ckv_api.hip", csrc / "ckv_select.hip", csrc / "ckv_decode.hip", csrc / "ckv_gather.hip", HERE / "emulator.cpp"):
        objs.append(str(pathlib.Path(where) / (src.name + ".o")))
        procs.append(subprocess.Popen([CXX, "-x", "c++", "-std=c++17", "-O1", "-fPIC", "-w", "-fsanitize=bounds", "-fsanitize-trap=bounds",
                                       f"-I{HERE}", f"-I{ROOT / 'include'}", f"-I{csrc}", "-c", str(src), "-o", objs[-1]]))
    assert [p.wait() for p in procs] == [0] * len(procs)
    lib = str(pathlib.Path(where) / "libckv_cpu.so")
    subprocess.run([CXX, "-shared", "-fPIC", *objs, "-o", lib], check=True)
    return lib


def load(path):
    """ctypes library; entry points whose kernels are not part of this build stay unresolved."""
    lib = ctypes.CDLL(path, mode=os.RTLD_LAZY)
    lib.ckv_workspace_bytes.restype = lib.ckv_decode_workspace_bytes.restype = ctypes.c_size_t
    lib.emu_set_hook.argtypes = [HOOK]
    return lib


def ptr(a):
    return None if a is None else ctypes.c_void_p(a.ctypes.data)


_mapped = []   # fenced memory, kept for the process


def fenced(nbytes) -> np.ndarray:
    """Zeroed bytes whose last one is the last before a page without access (16-byte aligned where nbytes is)."""
    page = mmap.PAGESIZE
    pages = (nbytes + page - 1) // page
    m = mmap.mmap(-1, (pages + 1) * page)
    whole = np.frombuffer(m, np.uint8)
    libc = ctypes.CDLL(None, use_errno=True)
    assert libc.mprotect(ctypes.c_void_p(whole.ctypes.data + pages * page), ctypes.c_size_t(page), 0) == 0
    _mapped.append(m)
    return whole[pages * page - nbytes:pages * page]


def aligned(nbytes, to=256) -> np.ndarray:
    raw = np.zeros(nbytes + to, np.uint8)
    off = -raw.ctypes.data % to
    return raw[off:off + nbytes]
