"""Counts what a call launches, by capturing it (nothing is replayed)."""
import ctypes
import re

import torch


def _hip():
    """The HIP runtime that this process has loaded."""
    return ctypes.CDLL(re.findall(r"\S*/libamdhip64\S*", open("/proc/self/maps").read())[0])


def launches(stream, call):
    """Nodes (launches and copies) of call(), which goes to the torch stream given and has run once before."""
    hip, graph, n = _hip(), ctypes.c_void_p(), ctypes.c_size_t()
    stream.synchronize()
    handle = ctypes.c_void_p(stream.cuda_stream)
    assert hip.hipStreamBeginCapture(handle, 1) == 0  # thread local
    try:
        call()
    finally:
        ended = hip.hipStreamEndCapture(handle, ctypes.byref(graph))
    assert ended == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    torch.cuda.synchronize()
    return n.value
