import ctypes
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def repo_root():
    return ROOT


class _KernelNode(ctypes.Structure):                 # hipKernelNodeParams
    _fields_ = [("block", ctypes.c_uint32 * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("grid", ctypes.c_uint32 * 3), ("args", ctypes.c_void_p), ("shared", ctypes.c_uint32)]


@pytest.fixture
def kernels_of():
    """kernels_of(run): the (mangled) names of the kernels that run() enqueues on the current stream, in order, from a
    captured graph that is never launched."""
    import torch
    from paper_2502_08923_amd import binding as cs

    def names(run):
        hip = cs.load_library()                       # (its own HIP runtime: symbols resolve through its dependencies)
        hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p
        hip.hipKernelNameRefByPtr.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
        graph = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(graph):
            run()
        handle, n = ctypes.c_void_p(graph.raw_cuda_graph()), ctypes.c_size_t()
        assert hip.hipGraphGetNodes(handle, None, ctypes.byref(n)) == 0
        nodes = (ctypes.c_void_p * n.value)()
        assert hip.hipGraphGetNodes(handle, nodes, ctypes.byref(n)) == 0
        out = []
        for node in nodes:
            kind, params = ctypes.c_int(), _KernelNode()
            assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0
            if kind.value == 0:                       # hipGraphNodeTypeKernel
                assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(params)) == 0
                out.append(hip.hipKernelNameRefByPtr(params.func, None).decode())
        return out

    return names
