"""Kernel sources compiled for the CPU, where every thread of a block is a
fiber: for what depends on the order in which blocks run, and for choices that
a kernel makes without leaving a trace in its results."""
import ctypes
import os
import subprocess

from paper_2601_01310_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
CLANG = os.path.join(os.path.dirname(os.path.dirname(build.HIPCC)), "llvm", "bin", "clang++")


def compile_host(name: str, out_dir) -> ctypes.CDLL:
    """Builds <name>.cpp into out_dir and loads it."""
    lib = os.path.join(str(out_dir), f"lib{name}.so")
    cmd = [CLANG, "-O1", "-std=c++17", "-fPIC", "-shared", "-w", f"-I{HERE}", f"-I{build.INCLUDE}",
           f"-I{build.CSRC}", os.path.join(HERE, name + ".cpp"), "-o", lib]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{' '.join(cmd)}\n{r.stderr}")
    return ctypes.CDLL(lib)
