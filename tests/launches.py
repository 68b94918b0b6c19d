"""The kernels that a call launches, in order, read from a graph that it is captured into."""
import ctypes as C
import re


class _Dim3(C.Structure):
    _fields_ = [("x", C.c_uint32), ("y", C.c_uint32), ("z", C.c_uint32)]


class _KernelNode(C.Structure):
    _fields_ = [("block", _Dim3), ("extra", C.c_void_p), ("func", C.c_void_p), ("grid", _Dim3), ("params", C.c_void_p), ("lds", C.c_uint32)]


def _runtime():
    """The HIP runtime that this process has loaded."""
    with open("/proc/self/maps") as f:
        path = next(m for m in (re.search(r"(/\S*libamdhip64\.so\S*)", line) for line in f) if m).group(1)
    lib = C.CDLL(path)
    lib.hipGraphGetNodes.argtypes = [C.c_void_p, C.c_void_p, C.POINTER(C.c_size_t)]
    lib.hipGraphNodeGetType.argtypes = [C.c_void_p, C.POINTER(C.c_int)]
    lib.hipGraphKernelNodeGetParams.argtypes = [C.c_void_p, C.POINTER(_KernelNode)]
    return lib


def launches(torch, call):
    """[(workgroups, threads each)] of the kernels of call(), which must be one that a graph can hold."""
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    stream = torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=stream):
        call()
    hip, raw, n = _runtime(), graph.raw_cuda_graph(), C.c_size_t(0)
    assert hip.hipGraphGetNodes(raw, None, C.byref(n)) == 0
    nodes = (C.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(raw, nodes, C.byref(n)) == 0
    out = []
    for node in nodes:
        kind, p = C.c_int(-1), _KernelNode()
        assert hip.hipGraphNodeGetType(node, C.byref(kind)) == 0 and kind.value == 0          # kernels only
        assert hip.hipGraphKernelNodeGetParams(node, C.byref(p)) == 0
        out.append((p.grid.x * p.grid.y * p.grid.z, p.block.x * p.block.y * p.block.z))
    return out
