"""Launch shapes of a call: its work is captured in a HIP graph, whose kernel
nodes are read and which is never run."""
import ctypes
import functools

import torch

_vp = ctypes.c_void_p


class _Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint32), ("y", ctypes.c_uint32), ("z", ctypes.c_uint32)]


class _KernelNodeParams(ctypes.Structure):  # hipKernelNodeParams
    _fields_ = [("block", _Dim3), ("extra", _vp), ("func", _vp), ("grid", _Dim3), ("params", _vp), ("shared", ctypes.c_uint32)]


@functools.lru_cache(None)
def _hip():
    """The HIP runtime this process already uses."""
    with open("/proc/self/maps") as f:
        paths = {line.split()[-1] for line in f if "libamdhip64" in line}
    assert len(paths) == 1, paths
    return ctypes.CDLL(paths.pop())


def _ok(status):
    assert status == 0, f"HIP error {status}"


def kernel_launches(call):
    """[((grid x, y), block x)] of the kernels that call(stream) launches, in no particular order."""
    hip = _hip()
    stream = torch.cuda.Stream()
    graph = _vp()
    _ok(hip.hipStreamBeginCapture(_vp(stream.cuda_stream), 1))  # thread-local mode
    try:
        call(stream)
    finally:
        _ok(hip.hipStreamEndCapture(_vp(stream.cuda_stream), ctypes.byref(graph)))
    n = ctypes.c_size_t()
    _ok(hip.hipGraphGetNodes(graph, None, ctypes.byref(n)))
    nodes = (_vp * n.value)()
    _ok(hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)))
    out = []
    for node in nodes:
        kind = ctypes.c_int()
        _ok(hip.hipGraphNodeGetType(_vp(node), ctypes.byref(kind)))
        if kind.value == 0:  # hipGraphNodeTypeKernel
            p = _KernelNodeParams()
            _ok(hip.hipGraphKernelNodeGetParams(_vp(node), ctypes.byref(p)))
            out.append(((p.grid.x, p.grid.y), p.block.x))
    _ok(hip.hipGraphDestroy(graph))
    return out
