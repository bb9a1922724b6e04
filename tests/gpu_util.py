"""Helpers for the GPU parity tests: host <-> device conversion and the error metric."""
import ctypes

import numpy as np
import torch

import workloads as W
from oracle import layer as L

DEV = "cuda:0"


def tdtype(dtype):
    return {W.FP32: torch.float32, W.FP16: torch.float16}.get(dtype, torch.bfloat16)


def to_dev(a, dtype):
    """numpy array (values already representable in the storage type) -> device tensor."""
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(DEV).to(tdtype(dtype)).contiguous()


def to_np(t):
    return t.detach().float().cpu().numpy().astype(np.float64)


def store(a, dtype):
    """Round host values to the storage type (returns fp32 numpy)."""
    a = np.asarray(a, dtype=np.float32)
    if dtype == W.FP16:
        return a.astype(np.float16).astype(np.float32)
    return W.round_to_bf16(a) if dtype == W.BF16 else a


def err(got, ref):
    return L.max_rel_err(to_np(got) if isinstance(got, torch.Tensor) else got, ref)


# fp16 keeps 3 more mantissa bits than bf16 (2^-11 against 2^-8 per rounding): an eighth of the bf16 bar, doubled
TOL = {W.FP32: 1e-4, W.BF16: 2e-2, W.FP16: 2.5e-3}


class _KernelNode(ctypes.Structure):   # hipKernelNodeParams
    _fields_ = [("block", ctypes.c_uint32 * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", ctypes.c_uint32 * 3),
                ("args", ctypes.c_void_p), ("shared", ctypes.c_uint32)]


def captured(step, grids=False, names=False):
    """(nodes, edges) of the graph that `step` is captured as, or the grids or (mangled) names of its kernels; nothing of it is run."""
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        step()
    with open("/proc/self/maps") as f:
        hip = ctypes.CDLL(next(l.split()[-1] for l in f if "libamdhip64" in l))
    raw, nodes, edges = ctypes.c_void_p(graph.raw_cuda_graph()), ctypes.c_size_t(0), ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(raw, None, ctypes.byref(nodes)) == 0 and nodes.value > 0
    assert hip.hipGraphGetEdges(raw, None, None, ctypes.byref(edges)) == 0
    if not grids and not names:
        return nodes.value, edges.value
    hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    each, out = (ctypes.c_void_p * nodes.value)(), []
    assert hip.hipGraphGetNodes(raw, each, ctypes.byref(nodes)) == 0
    for n in each:
        kind, k = ctypes.c_int(-1), _KernelNode()
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(n), ctypes.byref(kind)) == 0
        if kind.value == 0:   # hipGraphNodeTypeKernel
            assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(n), ctypes.byref(k)) == 0
            out.append(hip.hipKernelNameRefByPtr(ctypes.c_void_p(k.func), None).decode() if names else tuple(k.grid))
    return out


def shared_launches(step):
    """How many launches of several products of 256x256 tiles `step` makes."""
    return sum("gemm_bf16_products_kernel" in name for name in captured(step, names=True))


def branches(step):
    """How often the work that `step` enqueues leaves the caller's stream and comes back: captured, the edges beyond a chain's.
    Backward with every weight gradient on the helper stream: 3 (one per fork but the first); with the gradients in the
    launches of the data gradients and only that of the output projection there: 1."""
    step()                                          # (first-call set-up stays outside the capture)
    torch.cuda.synchronize()
    nodes, edges = captured(step)
    assert nodes > 1
    return edges - (nodes - 1)


def forks(step):
    return branches(step) != 0
