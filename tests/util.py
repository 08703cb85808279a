"""Helpers shared by the GPU parity tests: host<->device marshalling and the tolerance rule."""
import ctypes

import numpy as np
import torch

TORCH_DT = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
# relative tolerance of convolution outputs against the fp64 oracle: 1e-4 for fp32 and 2e-2 for
# bf16 are the stated targets; fp16 (11-bit significand, unit roundoff 2^-11 = 4.9e-4, one
# rounding of the output plus fp32 accumulation) gets 4e-3.
CONV_TOL = {"f32": 1e-4, "bf16": 2e-2, "f16": 4e-3}


class _KernelNode(ctypes.Structure):             # hipKernelNodeParams
    _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", ctypes.c_uint * 3),
                ("params", ctypes.c_void_p), ("lds", ctypes.c_uint)]


def kernels(fn):
    """The (mangled) names of the kernels that fn() launches, in order: the nodes of a graph that holds it."""
    import paper_1801_02108_amd as sb
    hip = sb.lib()
    hip.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    fn()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        fn()
    graph, n = ctypes.c_void_p(g.raw_cuda_graph()), ctypes.c_size_t()
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    names = []
    for node in nodes:
        kind, node = ctypes.c_int(), ctypes.c_void_p(node)
        assert hip.hipGraphNodeGetType(node, ctypes.byref(kind)) == 0 and kind.value == 0, "not a kernel"
        q = _KernelNode()
        assert hip.hipGraphKernelNodeGetParams(node, ctypes.byref(q)) == 0
        names.append(hip.hipKernelNameRefByPtr(ctypes.c_void_p(q.func), None).decode())
    return names


def template_args(name):
    """The whole-number and boolean template arguments in a kernel's mangled name: _ZN5sbnet6kernelILi1ELb0EE... -> (1, 0)."""
    import re
    m = re.search(r"I((?:L[ib]\d+E)+)E", name)
    return tuple(int(v) for v in re.findall(r"L[ib](\d+)E", m.group(1))) if m else ()


def to_dev(a, dtype):
    """numpy float array holding values exact in `dtype` -> contiguous device tensor of that dtype."""
    t = torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(TORCH_DT[dtype])
    return t.cuda().contiguous()


def to_host(t):
    """device tensor -> float64 numpy (exact)."""
    return t.detach().to(torch.float64).cpu().numpy()


def round_like(a64, dtype):
    """Round an fp64 array to the storage type the way the GPU's final store does (nearest even)."""
    return torch.from_numpy(np.ascontiguousarray(a64)).to(TORCH_DT[dtype]).to(torch.float64).numpy()


def assert_close(got, ref, tol, what=""):
    """|got - ref| <= tol*|ref| + tol*RMS(ref), element by element."""
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    assert got.shape == ref.shape, (got.shape, ref.shape)
    rms = float(np.sqrt(np.mean(ref * ref))) if ref.size else 0.0
    err = np.abs(got - ref)
    bound = tol * np.abs(ref) + tol * rms
    bad = err > bound
    if bad.any():
        k = np.unravel_index(np.argmax(err - bound), err.shape)
        raise AssertionError("%s: %d of %d elements out of tolerance %g; worst at %s got %r ref %r (rms %g)" % (
            what, int(bad.sum()), err.size, tol, k, got[k], ref[k], rms))
    return float(err.max() / (np.abs(ref).max() + 1e-300)) if ref.size else 0.0
