"""The kernels that a call launches, by recording it into a graph."""
import ctypes

import torch


class _Params(ctypes.Structure):
    _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", ctypes.c_uint * 3),
                ("params", ctypes.c_void_p), ("shared", ctypes.c_uint)]


class _Attributes(ctypes.Structure):
    _fields_ = [("binary", ctypes.c_int), ("cache", ctypes.c_int), ("constant", ctypes.c_size_t), ("local", ctypes.c_size_t), ("dynamic", ctypes.c_int),
                ("threads", ctypes.c_int), ("registers", ctypes.c_int), ("carveout", ctypes.c_int), ("ptx", ctypes.c_int), ("shared", ctypes.c_size_t)]


def kernels_of(call):
    """(name, bytes of private memory per thread, workgroups that a compute unit takes) of every kernel that call() launches on the current stream."""
    with open("/proc/self/maps") as maps:
        hip = ctypes.CDLL(next(line.split()[-1] for line in maps if "libamdhip64.so" in line))
    hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    hip.hipKernelNameRefByPtr.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        call()                                            # scratch of the stream
        stream.synchronize()
        graph, count = ctypes.c_void_p(), ctypes.c_size_t()
        assert hip.hipStreamBeginCapture(ctypes.c_void_p(stream.cuda_stream), 2) == 0
        call()
        assert hip.hipStreamEndCapture(ctypes.c_void_p(stream.cuda_stream), ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(count)) == 0
    nodes = (ctypes.c_void_p * count.value)()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(count)) == 0
    kernels = []
    for node in nodes:
        at, attributes = _Params(), _Attributes()
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(at)) == 0
        assert hip.hipFuncGetAttributes(ctypes.byref(attributes), ctypes.c_void_p(at.func)) == 0
        blocks, threads = ctypes.c_int(), at.block[0] * at.block[1] * at.block[2]
        assert hip.hipOccupancyMaxActiveBlocksPerMultiprocessor(ctypes.byref(blocks), ctypes.c_void_p(at.func), threads, ctypes.c_size_t(at.shared)) == 0
        kernels.append((hip.hipKernelNameRefByPtr(at.func, None).decode(), attributes.local, blocks.value))
    assert hip.hipGraphDestroy(graph) == 0
    return kernels
