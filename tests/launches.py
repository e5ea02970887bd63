"""Which kernels a call launches, read from a captured graph (that is never run): for tests that are about one kernel among several that give the same bits."""
import ctypes

import torch


class _KernelNode(ctypes.Structure):           # hipKernelNodeParams
    _fields_ = [("block", ctypes.c_uint32 * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", ctypes.c_uint32 * 3),
                ("args", ctypes.c_void_p), ("lds", ctypes.c_uint32)]


def _runtime():
    """The HIP runtime that is loaded already."""
    with open("/proc/self/maps") as f:
        paths = {line.split()[-1] for line in f if "libamdhip64.so" in line}
    assert len(paths) == 1, paths
    hip = ctypes.CDLL(paths.pop())
    hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    hip.hipKernelNameRefByPtr.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    hip.hipGraphGetNodes.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.POINTER(ctypes.c_size_t)]
    hip.hipGraphNodeGetType.argtypes = [ctypes.c_void_p, ctypes.POINTER(ctypes.c_int)]
    hip.hipGraphKernelNodeGetParams.argtypes = [ctypes.c_void_p, ctypes.POINTER(_KernelNode)]
    return hip


def launches(call, stream):
    """[(kernel name, workgroups, LDS bytes)] of what call() launches on `stream`."""
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        call()
    hip, count = _runtime(), ctypes.c_size_t()
    raw = graph.raw_cuda_graph()
    assert hip.hipGraphGetNodes(raw, None, ctypes.byref(count)) == 0
    nodes = (ctypes.c_void_p * count.value)()
    assert hip.hipGraphGetNodes(raw, nodes, ctypes.byref(count)) == 0
    found = []
    for node in nodes:
        kind, at = ctypes.c_int(), _KernelNode()
        assert hip.hipGraphNodeGetType(node, ctypes.byref(kind)) == 0
        if kind.value != 0:                    # hipGraphNodeTypeKernel
            continue
        assert hip.hipGraphKernelNodeGetParams(node, ctypes.byref(at)) == 0
        found.append((hip.hipKernelNameRefByPtr(at.func, None).decode(), at.grid[0] * at.grid[1] * at.grid[2], at.lds))
    return found
