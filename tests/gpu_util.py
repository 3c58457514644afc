"""Helpers of the GPU tests: host <-> device transfers of uint64 residue arrays, and
the kernels that a call launches."""
import ctypes
import re
from typing import NamedTuple

import numpy as np
import torch


def dev(a: np.ndarray) -> torch.Tensor:
    """uint64 numpy array -> int64 device tensor with the same bits."""
    a = np.ascontiguousarray(a, dtype=np.uint64)
    return torch.from_numpy(a.view(np.int64)).to("cuda")


def host(t: torch.Tensor) -> np.ndarray:
    torch.cuda.synchronize()
    return t.cpu().numpy().view(np.uint64)


def empty(shape) -> torch.Tensor:
    return torch.empty(shape, dtype=torch.int64, device="cuda")


def first_mismatch(a: np.ndarray, b: np.ndarray):
    """Index and values of the first differing element, or None."""
    if a.shape != b.shape:
        return ("shape", a.shape, b.shape)
    diff = np.argwhere(a != b)
    if len(diff) == 0:
        return None
    idx = tuple(int(v) for v in diff[0])
    return (idx, int(a[idx]), int(b[idx]), int(len(diff)))


class _KernelNodeParams(ctypes.Structure):  # hipKernelNodeParams
    _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("grid", ctypes.c_uint * 3), ("args", ctypes.c_void_p), ("lds", ctypes.c_uint)]


class _FuncAttributes(ctypes.Structure):  # hipFuncAttributes
    _fields_ = [("binaryVersion", ctypes.c_int), ("cacheModeCA", ctypes.c_int), ("constSizeBytes", ctypes.c_size_t),
                ("localSizeBytes", ctypes.c_size_t), ("maxDynamicSharedSizeBytes", ctypes.c_int),
                ("maxThreadsPerBlock", ctypes.c_int), ("numRegs", ctypes.c_int),
                ("preferredShmemCarveout", ctypes.c_int), ("ptxVersion", ctypes.c_int),
                ("sharedSizeBytes", ctypes.c_size_t)]


class Launch(NamedTuple):
    name: str      # kernel, without namespace and template arguments
    args: tuple    # its template arguments (numbers and 0 / 1 for false / true)
    grid: tuple
    block: tuple
    scratch: int   # scratch memory of a lane, bytes


def kernel_launches(call):
    """The kernels that call(stream) enqueues, in order, read from a graph captured of it
    (call(stream) runs once eagerly before)."""
    import paper_2603_16692_amd as ks
    hip = ks.HipEvents.runtime()
    hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    stream = torch.cuda.Stream()
    call(stream)
    stream.synchronize()
    s, graph, n = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t()
    assert hip.hipStreamBeginCapture(s, 1) == 0  # thread-local mode
    try:
        call(stream)
    finally:
        assert hip.hipStreamEndCapture(s, ctypes.byref(graph)) == 0
    try:
        assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
        nodes = (ctypes.c_void_p * n.value)()
        assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
        out = []
        for node in nodes:
            kind = ctypes.c_int()
            assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0
            if kind.value != 0:  # hipGraphNodeTypeKernel
                continue
            p, a = _KernelNodeParams(), _FuncAttributes()
            assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
            assert hip.hipFuncGetAttributes(ctypes.byref(a), ctypes.c_void_p(p.func)) == 0
            mangled = hip.hipKernelNameRefByPtr(ctypes.c_void_p(p.func), s).decode()
            name, args = re.search(r"(k_[a-z0-9_]+)(I(?:L[ib]\d+E)+E)?", mangled).groups()
            out.append(Launch(name, tuple(int(v) for v in re.findall(r"L[ib](\d+)E", args or "")),
                              tuple(p.grid), tuple(p.block), a.localSizeBytes))
        return out
    finally:
        hip.hipGraphDestroy(graph)
