"""The launch of the state pass: which workgroups the rule on the number of
(batch, head) states picks, read from the kernel nodes of a captured call.  An
in-place final state rules out sharing a slice's output rows between workgroups,
and must not take two slices a workgroup while one each fits the CUs."""

import ctypes
import functools

import pytest
import torch

import paper_2606_06034_amd as G

pytestmark = pytest.mark.gpu


class NodeParams(ctypes.Structure):  # hipKernelNodeParams
    _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("grid", ctypes.c_uint * 3), ("params", ctypes.c_void_p),
                ("shared", ctypes.c_uint)]


@functools.lru_cache(None)
def hip():
    """The HIP runtime this process has loaded."""
    with open("/proc/self/maps") as f:
        path = next(l.split()[-1] for l in f if "libamdhip64.so" in l)
    return ctypes.CDLL(path)


def launches(fn):
    """(workgroups, threads) of the kernels that fn launches."""
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        fn()
    graph = ctypes.c_void_p(g.raw_cuda_graph())
    n = ctypes.c_size_t()
    assert hip().hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip().hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    out = []
    for x in nodes:
        kind, p = ctypes.c_int(), NodeParams()
        assert hip().hipGraphNodeGetType(ctypes.c_void_p(x), ctypes.byref(kind)) == 0
        if kind.value == 0:  # a kernel
            assert hip().hipGraphKernelNodeGetParams(ctypes.c_void_p(x), ctypes.byref(p)) == 0
            out.append((p.grid[0] * p.grid[1] * p.grid[2], p.block[0] * p.block[1] * p.block[2]))
    return out


# (type, C, dk, dv, heads, in place): workgroups a group of 8 heads; head counts
# as shares of the 256 CUs (dv = 128: 8 slices a head)
CASES = [("bf16", 64, 128, 128, 4, False, 128), ("bf16", 64, 128, 128, 4, True, 64),
         ("bf16", 64, 128, 128, 16, True, 64), ("bf16", 64, 128, 128, 32, False, 64),
         ("bf16", 64, 128, 128, 32, True, 64), ("bf16", 64, 128, 128, 40, True, 32),
         ("bf16", 32, 128, 128, 32, False, 64), ("bf16", 32, 128, 128, 40, False, 32),
         ("bf16", 16, 128, 128, 8, False, 64), ("bf16", 16, 64, 64, 40, False, 32),
         ("f32", 64, 128, 128, 16, False, 128), ("f32", 64, 128, 128, 16, True, 64),
         ("f32", 64, 128, 128, 40, False, 32), ("f32", 64, 64, 128, 40, False, 64),
         ("f32", 16, 128, 128, 40, False, 32), ("f32", 16, 128, 128, 72, False, 64)]


@pytest.mark.parametrize("dt,C,dk,dv,H,in_place,per8", CASES)
def test_workgroups_of_the_state_pass(dt, C, dk, dv, H, in_place, per8):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the head counts are for 256 compute units")
    t = dict(device="cuda", dtype=torch.bfloat16 if dt == "bf16" else torch.float32)
    L = 2 * C
    Q, K, V = (torch.zeros((1, L, H, d), **t) for d in (dk, dk, dv))
    beta = torch.zeros((1, L, H), device="cuda")
    S0 = torch.zeros((1, H, dk, dv), device="cuda")
    Sf = S0 if in_place else torch.zeros_like(S0)
    O = torch.empty_like(V)
    ws = torch.empty(G.gdn_chunk_forward_workspace(1, L, H, dk, dv, C, K.dtype),
                     dtype=torch.uint8, device="cuda")
    call = lambda: G.gdn_chunk_forward(Q, K, V, beta, beta, C, S0=S0, O=O, S_final=Sf,
                                       workspace=ws)
    call()
    ks = launches(call)
    print(dt, C, dk, dv, H, in_place, ks, flush=True)
    assert len(ks) == 2 and ks[0] == (2 * H, 64)
    assert ks[1][0] == (H + 7) // 8 * per8
