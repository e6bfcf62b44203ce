"""The number of nodes of the HIP graph that a call records: its kernel launches, seen from outside."""
import ctypes


def nodes_of(call):
    import torch
    call()                                   # not the first call: nothing is set up while capturing
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    hip = ctypes.CDLL("libamdhip64.so")
    n = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value
