"""The kernels that a call enqueues, read from a captured graph of it."""
import ctypes

import torch

from paper_2601_17261_amd import binding


class _KernelNodeParams(ctypes.Structure):
    _fields_ = [("block", ctypes.c_uint32 * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", ctypes.c_uint32 * 3),
                ("params", ctypes.c_void_p), ("shared", ctypes.c_uint32)]


def kernels(stream, call):
    """(mangled names of the kernels in no particular order, node count) of call() on `stream`, its workspaces being reserved already"""
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        call()
    lib, raw = binding.load(), ctypes.c_void_p(graph.raw_cuda_graph())
    lib.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    lib.hipKernelNameRefByPtr.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    count = ctypes.c_size_t(0)
    assert lib.hipGraphGetNodes(raw, None, ctypes.byref(count)) == 0
    nodes = (ctypes.c_void_p * count.value)()
    assert lib.hipGraphGetNodes(raw, nodes, ctypes.byref(count)) == 0
    names = []
    for node in nodes:
        kind, p = ctypes.c_int(-1), _KernelNodeParams()
        assert lib.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0
        if kind.value == 0:          # a kernel
            assert lib.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
            names.append(lib.hipKernelNameRefByPtr(p.func, None).decode())
    return names, count.value
