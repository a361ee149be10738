"""Helpers shared by the GPU parity tests."""
import numpy as np
import torch


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    return t.detach().cpu().numpy()


def words(t):
    """Packed int32 tensor -> uint32 numpy."""
    return host(t).view(np.uint32)


def gpu_available():
    return torch.cuda.is_available()


def launches(call, side=None):
    """How many kernels `call` enqueues: the nodes of a graph that captures it, on a stream of its own or `side` (nothing of it runs)."""
    import ctypes
    from paper_1805_10111_amd import api
    g, side = torch.cuda.CUDAGraph(keep_graph=True), side or torch.cuda.Stream()
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            call()
    n = ctypes.c_size_t(0)
    assert api._lib.hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value
