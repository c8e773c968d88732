"""Which kernels a call launches."""
import ctypes
import re

import torch


class KernelNode(ctypes.Structure):                                      # hipKernelNodeParams
    _fields_ = [("block", ctypes.c_uint32 * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", ctypes.c_uint32 * 3),
                ("params", ctypes.c_void_p), ("lds", ctypes.c_uint32)]


def kernels(call):
    """The kernels of this library that a call launches, as (name, its numbers and flags): the nodes of its graph."""
    call()
    torch.cuda.synchronize()
    graph, count = torch.cuda.CUDAGraph(keep_graph=True), ctypes.c_size_t()
    with torch.cuda.graph(graph):
        call()
    with open("/proc/self/maps") as maps:
        hip = ctypes.CDLL(next(line.split()[-1] for line in maps if "libamdhip64" in line))
    hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    handle = ctypes.c_void_p(graph.raw_cuda_graph())
    assert hip.hipGraphGetNodes(handle, None, ctypes.byref(count)) == 0
    nodes = (ctypes.c_void_p * count.value)()
    assert hip.hipGraphGetNodes(handle, nodes, ctypes.byref(count)) == 0
    found = []
    for node in nodes:
        kind, params = ctypes.c_int(-1), KernelNode()
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0
        if kind.value != 0:                                              # hipGraphNodeTypeKernel
            continue
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(params)) == 0
        name = hip.hipKernelNameRefByPtr(ctypes.c_void_p(params.func), None).decode()
        own = re.search(r"\d+([a-z_]+_kernel)(I\w*)?", name)
        if "_GLOBAL__N_1" in name and own:
            found.append((own.group(1), tuple(int(x) for x in re.findall(r"L[ib](\d+)E", own.group(2) or ""))))
    return found
