"""csrc/stream_rule.h (which form a grouped GEMM of few rows takes) built for the host, so that tests know which form they reach."""
import collections
import ctypes
import functools
import os
import shutil
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2605_23764_amd", "csrc")
CXX = next((c for c in (shutil.which("g++"), shutil.which("clang++"), "/opt/rocm/llvm/bin/clang++") if c and os.path.exists(c)), None)

Form = collections.namedtuple("Form", "cols rows items whole")


@functools.lru_cache(maxsize=None)
def library():
    with tempfile.TemporaryDirectory() as tmp:
        so = os.path.join(tmp, "stream_rule.so")
        subprocess.run([CXX, "-std=c++17", "-O2", "-Wall", "-Werror", "-fPIC", "-shared", "-I", CSRC, os.path.join(HERE, "stream_rule.cpp"),
                        "-o", so], check=True)
        return ctypes.CDLL(so)


def form(max_rows, n_act, N, swiglu, G):
    """Form of a launch of G workgroups, or None where the stream does not take it."""
    if not library().stream_takes(max_rows, n_act, N, int(swiglu), G):
        return None
    out = (ctypes.c_int * 4)()
    library().stream_form(max_rows, n_act, N, int(swiglu), G, out)
    return Form(*out)


def faults(G):
    """Number of launches whose form cannot hold them, and one of them (max_rows, n_act, N, swiglu)."""
    first = (ctypes.c_int * 4)()
    return library().stream_faults(G, first), tuple(first)


def longer(G):
    """Number of launches with longer rounds than items of 128 columns throughout would have, and one of them."""
    first = (ctypes.c_int * 4)()
    return library().stream_longer(G, first), tuple(first)
