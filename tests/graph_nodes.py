"""What a call enqueues: the nodes of a HIP graph it is captured into."""
import ctypes
import os

import torch

from paper_2504_12526_amd import binding

KERNEL, MEMCPY = 0, 1


def hip():
    """The HIP runtime that torch and the library share."""
    binding.lib()
    paths = {line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line}
    assert len(paths) == 1, paths
    return ctypes.CDLL(os.path.realpath(paths.pop()))


def node_types(call):
    """Types of the nodes that call(stream) enqueues, in the order the runtime lists them; nothing is run."""
    h, vp = hip(), ctypes.c_void_p
    stream = torch.cuda.Stream()
    graph, n = vp(), ctypes.c_size_t()
    assert h.hipStreamBeginCapture(vp(stream.cuda_stream), 0) == 0               # global, as torch captures
    try:
        call(stream)
    finally:
        assert h.hipStreamEndCapture(vp(stream.cuda_stream), ctypes.byref(graph)) == 0
    assert h.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    nodes = (vp * n.value)()
    assert h.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    types = []
    for node in nodes:
        t = ctypes.c_int()
        assert h.hipGraphNodeGetType(vp(node), ctypes.byref(t)) == 0
        types.append(t.value)
    assert h.hipGraphDestroy(graph) == 0
    return types
