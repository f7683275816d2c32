"""Helpers for the GPU parity tests: move seeded storage arrays to the GPU
and compare with the oracle."""
import numpy as np
import torch

from oracle.stmoe_oracle import decode_storage
from paper_2606_15453_amd import workload as W

DEV = "cuda:0"


def to_dev(a: np.ndarray) -> torch.Tensor:
    """Storage array (uint16 bf16 bits or float32) -> device tensor (bfloat16 or float32)."""
    a = np.ascontiguousarray(a)
    if a.dtype == np.uint16:
        return torch.from_numpy(a.view(np.int16)).to(DEV).view(torch.bfloat16)
    return torch.from_numpy(a.astype(np.float32)).to(DEV)


def i32(a) -> torch.Tensor:
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(DEV)


def rel_l2(got, ref) -> float:
    """Largest relative L2 error over the output rows (the last axis is the
    hidden dimension; every batch row must meet the bound on its own)."""
    got = np.asarray(got, np.float64)
    ref = np.asarray(ref, np.float64)
    H = ref.shape[-1]
    g, r = got.reshape(-1, H), ref.reshape(-1, H)
    err = np.linalg.norm(g - r, axis=1) / np.maximum(np.linalg.norm(r, axis=1), 1e-300)
    return float(err.max())


def storage_dtype(cfg):
    return 1 if cfg.dtype == "bf16" else 0


def blob_dev(cfg, l, e, shared=False) -> torch.Tensor:
    dt = torch.bfloat16 if cfg.dtype == "bf16" else torch.float32
    out = torch.empty(cfg.blob_elems, dtype=dt, device=DEV)
    W.expert_blob_torch(cfg, l, e, out, shared=shared)
    return out


def expert_f64(cfg, l, e, shared=False):
    return tuple(decode_storage(m) for m in W.expert_matrices(cfg, l, e, shared))


def ptr_array(ptrs) -> torch.Tensor:
    return torch.tensor([int(p) for p in ptrs], dtype=torch.int64, device=DEV)


def graph_launches(fn, stream):
    """The kernel launches of fn() on `stream`, captured and not run:
    [(workgroups, threads per workgroup)] in order."""
    import ctypes as C

    class Params(C.Structure):       # hipKernelNodeParams
        _fields_ = [("block", C.c_uint32 * 3), ("extra", C.c_void_p), ("func", C.c_void_p), ("grid", C.c_uint32 * 3),
                    ("params", C.c_void_p), ("shared", C.c_uint32)]

    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g, stream=stream):
        fn()
    with open("/proc/self/maps") as f:
        hip = C.CDLL(next(line.split()[-1] for line in f if "libamdhip64" in line))
    graph, n = C.c_void_p(g.raw_cuda_graph()), C.c_size_t(0)
    assert hip.hipGraphGetNodes(graph, None, C.byref(n)) == 0
    nodes = (C.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(graph, nodes, C.byref(n)) == 0
    out = []
    for node in nodes:
        p = Params()
        assert hip.hipGraphKernelNodeGetParams(C.c_void_p(node), C.byref(p)) == 0
        out.append((p.grid[0] * p.grid[1] * p.grid[2], p.block[0] * p.block[1] * p.block[2]))
    return out
