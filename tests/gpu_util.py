"""Helpers shared by the GPU parity tests: move a seeded workload to the device, open the
library handles, and build the oracle's view of the same arrays."""
from __future__ import annotations

import ctypes

import numpy as np
import torch

import oracle
import paper_2502_11490_amd as ann
from workloads import to_host


def open_handles(wl, flags_mlp: int = 0, validate: bool = True):
    """wl: dict from workloads.make_workload (tensors on any device).  Returns (graph, mlp, dev dict)."""
    dev = {}
    for key in ("emb", "adj", "users", "entries", "W_q", "L_q", "cap_q"):
        if key in wl:
            dev[key] = wl[key].to("cuda").contiguous()
    dtype = {torch.bfloat16: ann.ANN_BF16, torch.float16: ann.ANN_F16}.get(wl["emb"].dtype, ann.ANN_F32)
    g = ann.ann_graph_load(dev["adj"], dev["emb"], ann.ANN_VALIDATE if validate else 0)
    d_user = wl["users"].shape[1]
    m = ann.ann_mlp_load(wl["W"], wl["b"], wl["head_w"], d_user, dtype, flags_mlp)
    return g, m, dev


def oracle_mlp(wl_host) -> oracle.Mlp:
    return oracle.Mlp(wl_host["W"], wl_host["b"], wl_host["head_w"])


def host_view(wl):
    return to_host(wl)


def same_list_fraction(a: np.ndarray, b: np.ndarray) -> float:
    return float(np.mean(np.all(a == b, axis=1)))


class _KernelNode(ctypes.Structure):  # hipKernelNodeParams
    _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("grid", ctypes.c_uint * 3), ("params", ctypes.c_void_p), ("lds", ctypes.c_uint)]


class _FuncAttributes(ctypes.Structure):  # hipFuncAttributes
    _fields_ = [("version", ctypes.c_int), ("ca", ctypes.c_int), ("const", ctypes.c_size_t), ("scratch", ctypes.c_size_t),
                ("dynamic", ctypes.c_int), ("threads", ctypes.c_int), ("registers", ctypes.c_int), ("carveout", ctypes.c_int),
                ("ptx", ctypes.c_int), ("lds", ctypes.c_size_t)]


def captured_kernels(call):
    """The kernel launches that `call` enqueues, recorded into a HIP graph: (mangled name, workgroups, threads of one,
    registers and scratch bytes of a lane) each."""
    with open("/proc/self/maps") as f:  # the runtime that is loaded already
        hip = ctypes.CDLL(next(line.split()[-1] for line in f if "libamdhip64.so" in line))
    hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    handle, n = ctypes.c_void_p(graph.raw_cuda_graph()), ctypes.c_size_t()
    assert hip.hipGraphGetNodes(handle, None, ctypes.byref(n)) == 0
    nodes, kind, p, out = (ctypes.c_void_p * n.value)(), ctypes.c_int(), _KernelNode(), []
    assert hip.hipGraphGetNodes(handle, nodes, ctypes.byref(n)) == 0
    for node in nodes:
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0
        assert kind.value == 0, "a node that is not a kernel"
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
        name = hip.hipKernelNameRefByPtr(ctypes.c_void_p(p.func), None)
        attr = _FuncAttributes()
        assert hip.hipFuncGetAttributes(ctypes.byref(attr), ctypes.c_void_p(p.func)) == 0
        out.append((name.decode() if name else "", p.grid[0], p.block[0], attr.registers, attr.scratch))
    return out


def captured_launches(call):
    """(workgroups, threads of one) of each of them."""
    return [launch[1:3] for launch in captured_kernels(call)]
