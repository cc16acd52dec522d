"""The state pass picks its workgroups by the number of (batch, head) states
(one or two slices of value columns each, one or two workgroups sharing a
slice's output rows, and no sharing when the final state overwrites the
initial one).  Every choice runs the same products in the same order per head,
so the heads of a large call equal, bit for bit, the same heads run in small
calls; the small calls are checked against the float64 oracle (the parity
bounds of the layer forward, 1e-5 in fp32 and 2e-2 in bf16)."""

import numpy as np
import pytest
import torch

import workloads as wl
from oracle import gdn, varlen

import paper_2606_06034_amd as G

from test_gpu_forward import check, dev, dev32, host, layer_inputs, run_ref

pytestmark = pytest.mark.gpu


def call(Q, K, V, beta, g, S0, C, dt, in_place=False):
    s0 = dev32(S0)
    O, Sf = G.gdn_chunk_forward(dev(Q, dt), dev(K, dt), dev(V, dt), dev32(beta), dev32(g), C,
                                S0=s0, S_final=s0 if in_place else None)
    return host(O), host(Sf)


# dv / 16 slices a head on 256 CUs: dv = 128 changes shape past 16 and past 32
# heads, dv = 64 past 32 and past 64; 9 and 33 are not whole groups of 8 heads
@pytest.mark.parametrize("C,dk,dv,H,dt", [(64, 128, 128, 33, "bf16"), (64, 128, 64, 66, "bf16"),
                                          (32, 64, 128, 33, "bf16"), (16, 128, 128, 33, "bf16"),
                                          (64, 64, 64, 65, "f32"), (32, 128, 128, 18, "f32"),
                                          (16, 64, 64, 9, "f32")])
def test_every_workgroup_shape_gives_the_same_bits(C, dk, dv, H, dt):
    print(f"state pass shapes C={C} dk={dk} dv={dv} H={H} {dt}", flush=True)
    Q, K, V, beta, g, S0 = layer_inputs(C, dt, B=1, L=5 * C, H=H, dk=dk, dv=dv, seed=40 + H)
    O, Sf = call(Q, K, V, beta, g, S0, C, dt)
    Oi, Si = call(Q, K, V, beta, g, S0, C, dt, in_place=True)
    assert np.array_equal(Oi, O) and np.array_equal(Si, Sf)
    n = 3
    for cut in (n, 20, H):  # small, middle and full head counts, the last heads
        if cut > H:
            continue
        sl = slice(H - cut, H)
        o, s = call(Q[:, :, sl], K[:, :, sl], V[:, :, sl], beta[:, :, sl], g[:, :, sl], S0[:, sl],
                    C, dt)
        assert np.array_equal(o, O[:, :, sl]) and np.array_equal(s, Sf[:, sl]), cut
    sl = slice(H - n, H)
    Or, Sr = run_ref(Q[:, :, sl], K[:, :, sl], V[:, :, sl], beta[:, :, sl], g[:, :, sl],
                     S0[:, sl], C)
    check(O[:, :, sl], Or, dt, "O")
    check(Sf[:, sl], Sr, dt, "S_final")


@pytest.mark.parametrize("C,dt", [(64, "bf16"), (16, "bf16"), (64, "f32")])
@pytest.mark.parametrize("nseq", [2, 9, 19])
def test_packed_shapes(C, dt, nseq):
    # lengths around the chunk size: 1, C - 1, C, C + 1, several chunks, empty
    rng = np.random.default_rng(nseq)
    lengths = [[1, C - 1, C, C + 1, 3 * C + 5, 0, 2 * C][i % 7] for i in range(nseq)]
    print(f"packed state pass shapes C={C} {dt} {lengths}", flush=True)
    cu = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    T, H, d = int(cu[-1]), 2, 128
    z = rng.standard_normal((1, T, H, d))
    K = z / np.linalg.norm(z, axis=-1, keepdims=True)
    Q = 0.3 * rng.standard_normal((1, T, H, d))
    V = rng.standard_normal((1, T, H, d))
    rnd = wl.round_to_bf16 if dt == "bf16" else (lambda x: x)
    Q, K, V = (rnd(x.astype(np.float32)).astype(np.float64) for x in (Q, K, V))
    beta = rng.random((1, T, H)).astype(np.float32)
    g = varlen.varlen_cumsum(-0.1 * rng.random((T, H)), cu, C)[None].astype(np.float32)
    S0 = rng.standard_normal((nseq, H, d, d)).astype(np.float32)
    N, S = gdn.default_order(C)
    tables = G.gdn_varlen_tables(cu, C)
    args = (dev(Q, dt), dev(K, dt), dev(V, dt), dev32(beta), dev32(g))
    O, Sf = G.gdn_chunk_forward_varlen(*args, tables, C, S0=dev32(S0))
    s0 = dev32(S0)
    Oi, Si = G.gdn_chunk_forward_varlen(*args, tables, C, S0=s0, S_final=s0)
    assert torch.equal(O, Oi) and torch.equal(Sf, Si)
    Or, Sr = varlen.forward_varlen_chunked(Q, K, V, beta, g, cu, C, S0, d ** -0.5,
                                           inverse=lambda A: gdn.neumann_inverse(A, N, S))
    check(host(O), Or, dt, "O")
    check(host(Sf), Sr, dt, "S_final")


# fp32 past 256 slices: C = 64 as two slices with a ring of one chunk (dk = 128)
# or one slice with such a ring (dk = 64); C = 32 as two slices (dk = 128) or one
# with a ring of two; C = 16 as one slice from 512 (dk = 64: 256) to 640 slices
# and as two on either side
@pytest.mark.parametrize("C,dk,dv,H", [(64, 128, 128, 33), (64, 128, 64, 66), (64, 64, 128, 34),
                                       (32, 128, 64, 65), (32, 64, 128, 33), (16, 128, 128, 33),
                                       (16, 128, 128, 65), (16, 64, 128, 33), (16, 64, 128, 81)])
def test_fp32_shapes_past_the_compute_units(C, dk, dv, H):
    test_every_workgroup_shape_gives_the_same_bits(C, dk, dv, H, "f32")


@pytest.mark.parametrize("C,H", [(64, 19), (32, 9), (16, 9), (16, 42)])
def test_packed_fp32_shapes_past_the_compute_units(C, H):
    # ragged and empty sequences; the small call takes one slice a workgroup
    rng = np.random.default_rng(H)
    lengths, d = [2 * C + 1, 1, 0, C], 128
    cu = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    T = int(cu[-1])
    print(f"packed fp32 state pass C={C} H={H}", flush=True)
    z = rng.standard_normal((2, 1, T, H, d)).astype(np.float32)
    Q, K = z / np.linalg.norm(z, axis=-1, keepdims=True)
    V = rng.standard_normal((1, T, H, d)).astype(np.float32)
    beta = rng.random((1, T, H)).astype(np.float32)
    g = varlen.varlen_cumsum(-0.1 * rng.random((T, H)), cu, C)[None].astype(np.float32)
    S0 = rng.standard_normal((len(lengths), H, d, d)).astype(np.float32)
    tables = G.gdn_varlen_tables(cu, C)

    def part(sl):
        return G.gdn_chunk_forward_varlen(
            *(dev(x[:, :, sl], "f32") for x in (Q, K, V)), dev32(beta[:, :, sl]),
            dev32(g[:, :, sl]), tables, C, S0=dev32(S0[:, sl]))

    O, Sf = part(slice(0, H))
    o, s = part(slice(H - 2, H))
    assert torch.equal(O[:, :, H - 2:], o) and torch.equal(Sf[:, H - 2:], s)
    N, S = gdn.default_order(C)
    Or, Sr = varlen.forward_varlen_chunked(
        *(x[:, :, H - 2:].astype(np.float64) for x in (Q, K, V)), beta[:, :, H - 2:],
        g[:, :, H - 2:], cu, C, S0[:, H - 2:], d ** -0.5,
        inverse=lambda A: gdn.neumann_inverse(A, N, S))
    check(host(o), Or, "f32", "O")
    check(host(s), Sr, "f32", "S_final")
