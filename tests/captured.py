"""Which kernels a call launches: the call is recorded into a graph, and the graph's kernel nodes are read."""
from __future__ import annotations

import ctypes as C


class _Dim3(C.Structure):
    _fields_ = [("x", C.c_uint), ("y", C.c_uint), ("z", C.c_uint)]


class _KernelNodeParams(C.Structure):  # hipKernelNodeParams
    _fields_ = [("blockDim", _Dim3), ("extra", C.c_void_p), ("func", C.c_void_p), ("gridDim", _Dim3),
                ("kernelParams", C.c_void_p), ("sharedMemBytes", C.c_uint)]


def _runtime():
    with open("/proc/self/maps") as f:  # the one this process has loaded
        return C.CDLL(next(line.split()[-1] for line in f if "libamdhip64" in line))


def launches(call):
    """(mangled) names of the kernels that call() launches on torch's current stream, in order.  The call is
    recorded, not run."""
    import torch
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    hip, raw, n = _runtime(), C.c_void_p(graph.raw_cuda_graph()), C.c_size_t(0)
    hip.hipKernelNameRefByPtr.restype = C.c_char_p
    assert hip.hipGraphGetNodes(raw, None, C.byref(n)) == 0
    nodes = (C.c_void_p * max(n.value, 1))()
    assert hip.hipGraphGetNodes(raw, nodes, C.byref(n)) == 0
    names = []
    for node in nodes[:n.value]:
        kind, params = C.c_int(-1), _KernelNodeParams()
        assert hip.hipGraphNodeGetType(C.c_void_p(node), C.byref(kind)) == 0 and kind.value == 0, "a node that is no kernel"
        assert hip.hipGraphKernelNodeGetParams(C.c_void_p(node), C.byref(params)) == 0
        names.append(hip.hipKernelNameRefByPtr(C.c_void_p(params.func), None).decode())
    return names
