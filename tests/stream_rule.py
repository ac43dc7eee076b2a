"""csrc/stream_rule.h (which form a grouped GEMM of few rows takes) built for the host, so that tests know which form they reach."""
import collections
import ctypes

from host_build import CXX, library as _build  # noqa: F401  (CXX: None without a host compiler)

Form = collections.namedtuple("Form", "cols rows items whole")


def library():
    return _build("stream_rule.cpp")


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
