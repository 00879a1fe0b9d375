"""Helpers shared by the GPU tests: the kernel launches of a call, and how many of
a launch's workgroups a compute unit holds."""
import ctypes

import numpy as np
import torch


class KernelParams(ctypes.Structure):
    """hipKernelNodeParams."""
    _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("grid", ctypes.c_uint * 3), ("args", ctypes.c_void_p), ("lds", ctypes.c_uint)]


def _hip():
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64.so" in line)
    return ctypes.CDLL(path)


def launches(call):
    """The kernel launches of `call`, captured and not run."""
    hip, vp = _hip(), ctypes.c_void_p
    stream, graph, n = torch.cuda.Stream(), vp(), ctypes.c_size_t()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        assert hip.hipStreamBeginCapture(vp(stream.cuda_stream), 1) == 0  # (thread-local)
        try:
            call()
        finally:
            assert hip.hipStreamEndCapture(vp(stream.cuda_stream), ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    nodes = (vp * n.value)()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    out = []
    for node in nodes:
        p = KernelParams()
        assert hip.hipGraphKernelNodeGetParams(vp(node), ctypes.byref(p)) == 0
        out.append(p)
    assert hip.hipGraphDestroy(graph) == 0
    return out


def residency(p):
    """Workgroups of a launch that a compute unit holds."""
    n = ctypes.c_int()
    assert _hip().hipOccupancyMaxActiveBlocksPerMultiprocessor(ctypes.byref(n), ctypes.c_void_p(p.func),
                                                               int(np.prod(p.block)), ctypes.c_size_t(p.lds)) == 0
    return n.value
