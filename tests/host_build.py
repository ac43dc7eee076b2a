"""Parts of the kernels' sources that are free of device code, built for the host as a shared library."""
import ctypes
import functools
import os
import shutil
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2605_23764_amd", "csrc")
CXX = next((c for c in (shutil.which("g++"), shutil.which("clang++"), "/opt/rocm/llvm/bin/clang++") if c and os.path.exists(c)), None)


@functools.lru_cache(maxsize=None)
def library(source):
    """tests/<source>, which includes headers of csrc/."""
    with tempfile.TemporaryDirectory() as tmp:
        so = os.path.join(tmp, "host.so")
        subprocess.run([CXX, "-std=c++17", "-O2", "-Wall", "-Werror", "-fPIC", "-shared", "-I", CSRC, os.path.join(HERE, source), "-o", so],
                       check=True)
        return ctypes.CDLL(so)
