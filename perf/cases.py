"""Performance cases: the work users of this library have it do, through its
public entry points, over the range of sizes they use.

`listed()` names the cases, `draw(rng)` gives one more of the same ranges,
`prepare` makes a case's inputs on the GPU, `run` is one call (or the calls of
one step), `work` is what the computation cannot do without, `tolerance` says
how far another correct implementation may be off, and `exact` is the result in
64 bits from plain torch.

The paths:
  layer        the chunk-wise Gated DeltaNet layer forward over equal-length
               sequences, state in and out (prefill, chunked continuation)
  layer_packed the same over packed sequences of different lengths
  step         the layer forward without allocation (serving loops)
  wy           the fused build A -> inverse -> W, U step
  wy_packed    the same over packed sequences
  inverse      the standalone chunk inverse of given tiles
  int          A from K, quantised and inverted in integers, in one launch

Inputs follow the library's own workloads: unit-norm keys and queries, values
N(0, 1), beta = sigmoid(N(0, 1)), log-decay -softplus(x + s) per token.  The
heads of a trained layer range from fast- to slow-forgetting, so even heads
draw with s = 3 and odd heads with s = -4 ("mixed"); the integer paths use the
wide gates -softplus(2 x + 1) of the low-bit workload.
"""

import math
import random

import numpy as np
import torch

import paper_2606_06034_amd as G

_DT = {"bf16": torch.bfloat16, "f32": torch.float32}
_ORDER = {16: (3, 2), 32: (3, 4), 64: (3, 8), 128: (3, 8)}


def _case(name, path, **kw):
    c = dict(path=path, B=1, L=8192, H=16, dk=128, dv=128, C=64, dtype="bf16", mode="neumann",
             gate="mixed", mix=0, want_T=False, bits=0)
    c.update(kw)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest call: one 64-token chunk for each of four users of a
        # serving loop, state handed on, no allocation
        _case("step_64x4", "step", B=4, L=64),
        # the prompt of the Qwen3.5-shaped layer: 8192 tokens, 16 key heads
        _case("layer_prefill_8k", "layer"),
        # a serving batch of the same size: sequences of 1 to 4096 tokens packed
        _case("layer_packed_8k", "layer_packed", mix=3000),
        # long context: 131072 tokens, 32 heads, the largest layer call
        _case("layer_long_128k", "layer", L=131072, H=32),
        # the quantised layer: INT16 inverse inside the bf16 layer
        _case("layer_int16_8k", "layer", mode="int16"),
        # the layer in fp32 with the exact inverse, as used to check a model
        _case("layer_f32_1k", "layer", L=1024, H=4, dtype="f32", mode="exact"),
        # W and U alone (the step before a layer of the user's own), long context
        _case("wy_long_128k", "wy", L=131072, H=32),
        # the largest chunk size, a training-sized batch
        _case("wy_c128_64k", "wy", B=4, L=16384, H=32, C=128),
        # packed sequences, exact inverse, tiles wanted too
        _case("wy_packed_8k", "wy_packed", mix=3000, mode="exact", want_T=True),
        # the standalone inverse of a batch of tiles
        _case("inverse_c64_32k", "inverse", B=4, L=16384, H=32),
        # the low-bit inverses from K in one launch
        _case("int8_c64_32k", "int", B=4, L=16384, H=32, bits=8, gate="wide"),
        _case("int16_c64_32k", "int", B=4, L=16384, H=32, bits=16, gate="wide"),
    ]


def draw(rng):
    """One more case: sizes over the listed range (log-uniform), odd head and
    chunk counts, every chunk size, feature width, type and mode in use."""
    path = rng.choice(["layer", "layer", "layer", "layer_packed", "layer_packed", "step", "wy",
                       "wy", "wy_packed", "inverse", "inverse", "int", "int"])
    H = rng.choice([1, 2, 3, 4, 5, 6, 8, 12, 16, 20, 24, 32, 48])
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    dk, dv = rng.choice([(128, 128)] * 5 + [(64, 64), (128, 64), (64, 128)])
    layer = path in ("layer", "layer_packed", "step")
    C = rng.choice([64, 64, 64, 32, 16] if layer else [64, 64, 64, 32, 16, 128])
    cap = (1 << 20) // H  # tokens; token-heads stay below a quarter of the largest case's
    if dtype == "f32" or path == "int":
        cap //= 4
    if path == "step":
        cap = min(cap, 4096, 49152 // H)  # within the library's scratch in either type
    cap = max(C, min(cap, 65536 * C // 64))
    T = int(round(math.exp(rng.uniform(math.log(C), math.log(cap)))))
    B = rng.choice([1, 1, 1, 2, 3, 4, 7])
    mode = rng.choice(["neumann", "neumann", "neumann", "exact"])
    gate = rng.choice(["mixed", "mixed", "default"])
    kw = {}
    if layer and dk == dv == 128 and rng.random() < 0.25:
        mode = rng.choice(["int16", "int8"])
    if path == "inverse" and rng.random() < 0.25:
        mode = "fwdsub"
    if path == "int":
        kw = dict(bits=rng.choice([8, 16]))
        gate, mode = rng.choice(["wide", "default"]), "neumann"
    if path in ("wy", "wy_packed"):
        kw = dict(want_T=rng.random() < 0.3)
    if path.endswith("_packed"):
        B, L = 1, T
        kw["mix"] = rng.randrange(1, 1 << 30)
    else:
        L = C * max(1, T // (B * C))
    return _case(None, path, B=B, L=L, H=H, dk=dk, dv=dv, C=C, dtype=dtype, mode=mode, gate=gate,
                 **kw)


# ---------------------------------------------------------------------------
# inputs


def _lengths(case):
    """Sequence lengths: B equal ones, or a mix log-uniform in [1, 4096]."""
    if not case["path"].endswith("_packed"):
        return [case["L"]] * case["B"]
    rng, out, left = random.Random(case["mix"]), [], case["L"]
    while left > 0:
        n = min(left, int(math.exp(rng.uniform(0.0, math.log(4097.0)))))
        out.append(max(1, n))
        left -= out[-1]
    return out


def _chunks(case):
    """(first token of every chunk, its tokens, the sequence it belongs to)."""
    C, t, start, size, seq = case["C"], 0, [], [], []
    for s, n in enumerate(_lengths(case)):
        for a in range(0, n, C):
            start.append(t + a)
            size.append(min(C, n - a))
            seq.append(s)
        t += n
    return np.array(start), np.array(size), np.array(seq)


def _inputs(case, seed):
    """K, V, Q [1 or B, L, H, d], beta, g [.., L, H], S0 [nseq, H, dk, dv]."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 13)
    B, L, H, dk, dv, C = (case[k] for k in ("B", "L", "H", "dk", "dv", "C"))
    dt = _DT[case["dtype"]]

    def rnd(*shape):
        return torch.randn(shape, generator=gen, device="cuda")

    def unit(*shape):
        z = rnd(*shape)
        return z.div_(z.norm(dim=-1, keepdim=True)).to(dt)

    K = unit(B, L, H, dk)
    V = rnd(B, L, H, dv).to(dt)
    beta = torch.sigmoid(rnd(B, L, H))
    x = rnd(B, L, H).double()
    if case["gate"] == "wide":
        x = 2 * x + 1
    else:
        x = x + 3
        if case["gate"] == "mixed":
            x[..., 1::2] -= 7
    inc = -torch.nn.functional.softplus(x)
    if case["path"].endswith("_packed"):
        start, size, _ = _chunks(case)
        first = torch.from_numpy(np.repeat(start, size)).cuda()
        cs = torch.cat([torch.zeros_like(inc[:, :1]), inc.cumsum(1)], 1)
        g = (cs[:, 1:] - cs[:, first]).float()
    else:
        g = inc.view(B, L // C, C, H).cumsum(2).view(B, L, H).float()
    out = dict(K=K, V=V, beta=beta, g=g.contiguous())
    if case["path"] in ("layer", "layer_packed", "step"):
        out["Q"] = unit(B, L, H, dk)
        out["S0"] = rnd(len(_lengths(case)), H, dk, dv)
    return out


def _tiles(case, x):
    """A of every tile [B, H, L / C, C, C] for the standalone inverse."""
    return G.gdn_build_A(x["K"], x["beta"], x["g"], case["C"])


def prepare(case, seed):
    """The inputs, and for packed sequences their chunk tables; for the
    standalone inverse the tiles; for the serving step its output buffers."""
    x = _inputs(case, seed)
    x["case"] = case
    if case["path"].endswith("_packed"):
        cu = [0]
        for n in _lengths(case):
            cu.append(cu[-1] + n)
        x["tables"] = G.gdn_varlen_tables(cu, case["C"])
    if case["path"] == "inverse":
        x = dict(case=case, A=_tiles(case, x))
    if case["path"] == "step":
        x["O"] = torch.empty_like(x["V"])
        x["S_final"] = torch.empty_like(x["S0"])
    return x


def run(s):
    c = s["case"]
    path, C = c["path"], c["C"]
    N, S = _ORDER[C]
    if path == "layer":
        return G.gdn_chunk_forward(s["Q"], s["K"], s["V"], s["beta"], s["g"], C, S0=s["S0"],
                                   inverse=c["mode"])
    if path == "layer_packed":
        return G.gdn_chunk_forward_varlen(s["Q"], s["K"], s["V"], s["beta"], s["g"], s["tables"],
                                          C, S0=s["S0"], inverse=c["mode"])
    if path == "step":
        return G.gdn_chunk_forward_noalloc(s["Q"], s["K"], s["V"], s["beta"], s["g"], C, s["O"],
                                           S0=s["S0"], S_final=s["S_final"], inverse=c["mode"])
    if path == "wy":
        if c["mode"] == "exact":
            return G.gdn_chunk_wy_fused_blockwise(s["K"], s["V"], s["beta"], s["g"], C,
                                                  want_T=c["want_T"])
        return G.gdn_chunk_wy_fused(s["K"], s["V"], s["beta"], s["g"], C, N, S,
                                    want_T=c["want_T"])
    if path == "wy_packed":
        return G.gdn_chunk_wy_fused_varlen(s["K"], s["V"], s["beta"], s["g"], s["tables"], C,
                                           exact=c["mode"] == "exact", want_T=c["want_T"])
    if path == "inverse":
        if c["mode"] == "exact":
            return G.gdn_chunk_inverse_blockwise(s["A"])
        if c["mode"] == "fwdsub":
            return G.gdn_chunk_inverse_fwdsub(s["A"])
        return G.gdn_chunk_inverse_neumann(s["A"], N, S)
    f = G.gdn_chunk_inverse_neumann_i8_fused if c["bits"] == 8 else \
        G.gdn_chunk_inverse_neumann_i16_fused
    return f(s["K"], s["beta"], s["g"], C, N, S)


# ---------------------------------------------------------------------------
# what a pass cannot do without


def _inverse_flops(case):
    """Non-zero (lower-triangular) part of the method's products, per tile."""
    C = case["C"]

    def lower(n):  # product of two lower-triangular n x n matrices
        return n * (n + 1) * (n + 2) / 3

    if case["mode"] in ("exact", "fwdsub"):
        return (C ** 3 - C) / 3
    N, S = _ORDER[C]
    if C == 128:
        return 2 * (N + S) * lower(64) + 2 * 64 * 64 * 65
    return (N + S) * lower(C)


def work(case):
    """Each input read once, each output written once; the method's own
    products, counting the entries a triangular product can fill."""
    H, dk, dv, C, path = (case[k] for k in ("H", "dk", "dv", "C", "path"))
    es = 4 if case["dtype"] == "f32" else 2
    tok = case["B"] * case["L"] * H
    n = H * len(_chunks(case)[0])
    if path == "inverse":
        return {"bytes": 2 * n * C * C * es, "flops": n * _inverse_flops(case)}
    gram = n * C * C * dk
    if path == "int":
        nexp = 3 if C == 128 else 1
        return {"bytes": tok * (dk * es + 8) + n * (C * C * case["bits"] // 8 + 4 * nexp),
                "flops": gram + n * _inverse_flops(case) * (1 if case["bits"] == 8 else 4)}
    flops = gram + n * (_inverse_flops(case) + C * (C + 1) * (dk + dv))
    if path in ("wy", "wy_packed"):
        return {"bytes": tok * (2 * (dk + dv) * es + 8) + (n * C * C * es if case["want_T"] else 0),
                "flops": flops}
    nseq = len(_lengths(case))
    flops += n * (6 * C * dk * dv + C * (C + 1) * (dk + dv))
    return {"bytes": tok * ((2 * dk + 2 * dv) * es + 8) + 2 * nseq * H * dk * dv * 4,
            "flops": flops}


def tolerance(case):
    """Integer results are exact.  Elsewhere about four times the measured
    distance from the 64-bit result: bf16 rounds every operand of a product
    (layer 3.8e-3, W and U 2.4e-3, the inverse of small off-diagonals 2.9e-4),
    fp32 rounds the sums (2.5e-7); the integer inverses inside an fp32 layer
    carry their codes' rounding, and a code may round the other way."""
    if case["path"] == "int":
        return "exact"
    if case["dtype"] == "f32":
        if case["mode"] == "int8":
            return {"rel": 4e-3, "max": 0.1}
        if case["mode"] == "int16":
            return {"rel": 2e-5, "max": 1e-3}
        return {"rel": 1e-6, "max": 1e-4}
    if case["path"] == "inverse":
        return {"rel": 1.2e-3, "max": 0.05}
    if case["path"] in ("wy", "wy_packed"):
        return {"rel": 1e-2, "max": 0.15}
    return {"rel": 1.5e-2, "max": 0.2}


# ---------------------------------------------------------------------------
# the results in 64 bits


def _eye(A):
    return torch.eye(A.shape[-1], dtype=A.dtype, device=A.device)


def _inv64(A, N, S):
    """(I + A)^-1 of strictly lower tiles: T_hat(N, S), or exact (N None) by
    the finite product (I + L)(I + L^2)(I + L^4)..., L = -A."""
    I, L = _eye(A), -A
    if N is None:
        T, P, k = I + L, L, 1
        while 2 * k < A.shape[-1]:
            P = P @ P
            T = T + T @ P
            k *= 2
        return T
    i = torch.arange(A.shape[-1], device=A.device)
    keep = (i[:, None] - i[None, :] <= N).to(A.dtype)
    T0, P = I + (L if N >= 1 else 0), L
    for _ in range(2, N + 1):
        P = P @ L
        T0 = T0 + P
    T0 = T0 * keep
    E = I - (I + A) @ T0
    R = I + (E if S >= 1 else 0)
    P = E
    for _ in range(2, S + 1):
        P = P @ E
        R = R + P
    return T0 @ R


def _inverse64(A, case):
    C = case["C"]
    N, S = (None, None) if case["mode"] in ("exact", "fwdsub") else _ORDER[C]
    if C < 128:
        return _inv64(A, N, S)
    X11 = _inv64(A[..., :64, :64].contiguous(), N, S)
    X22 = _inv64(A[..., 64:, 64:].contiguous(), N, S)
    X21 = -(X22 @ A[..., 64:, :64].contiguous() @ X11)
    T = torch.zeros_like(A)
    T[..., :64, :64], T[..., 64:, :64], T[..., 64:, 64:] = X11, X21, X22
    return T


def exact(case, seed):
    path, C, H, dk, dv = (case[k] for k in ("path", "C", "H", "dk", "dv"))
    if path == "int":
        return None  # codes: no 64-bit counterpart
    x = _inputs(case, seed)
    if path == "inverse":
        return _inverse64(torch.tril(_tiles(case, x).double(), -1), case)
    start, size, seq = _chunks(case)
    nch, B, L = len(start), case["B"], case["L"]
    at = start[:, None] + np.minimum(np.arange(C)[None, :], size[:, None] - 1)
    at = torch.from_numpy(at).cuda()
    live = torch.from_numpy(np.arange(C)[None, :] < size[:, None]).cuda()  # [nch, C]

    def tiles(name):  # [nch, H, C, d] or [nch, H, C]; rows past the chunk's tokens repeat its last
        t = x[name].reshape((B * L,) + tuple(x[name].shape[2:]))[at]
        return t.transpose(1, 2).double().contiguous()

    lm = live[:, None, :].double()
    K, V = tiles("K") * lm[..., None], tiles("V") * lm[..., None]
    beta, g = tiles("beta") * lm, tiles("g")
    D = torch.tril(torch.exp((g[..., :, None] - g[..., None, :]).clamp(max=0.0)))
    KT = K.transpose(-1, -2).contiguous()
    A = torch.tril(beta[..., None] * (K @ KT) * D, -1)
    T = _inverse64(A, case)

    def rows(t, d):  # back to [B, L, H, d]
        out = torch.empty((B * L, H, d), dtype=torch.float64, device="cuda")
        out[at[live]] = t.transpose(1, 2)[live]
        return out.reshape(B, L, H, d)

    if path in ("wy", "wy_packed"):
        W, U = T @ (beta[..., None] * K), T @ (beta[..., None] * V)
        out = (rows(W, dk), rows(U, dv))
        if not case["want_T"]:
            return out
        Tt = T.transpose(0, 1).contiguous()  # [H, nch, C, C]
        if path == "wy":
            Tt = Tt.reshape(H, B, nch // B, C, C).transpose(0, 1).contiguous()
        return out + (Tt,)
    Q = tiles("Q")
    eg = torch.exp(g)[..., None]
    W, U = T @ (beta[..., None] * eg * K), T @ (beta[..., None] * V)
    P = (Q @ KT) * D
    Qg = eg * Q
    Kd = (torch.exp(g[..., -1:] - g)[..., None] * K).transpose(-1, -2).contiguous()
    el = torch.exp(g[..., -1])[..., None, None]
    del A, T, D, K, KT, V, Q
    S = x["S0"].double()
    O = torch.empty((nch, H, C, dv), dtype=torch.float64, device="cuda")
    scale = dk ** -0.5
    first = np.searchsorted(seq, np.arange(len(_lengths(case))))
    count = np.bincount(seq, minlength=len(first))
    for k in range(int(count.max())):
        run_on = np.nonzero(count > k)[0]
        s, c = torch.from_numpy(run_on).cuda(), torch.from_numpy(first[run_on] + k).cuda()
        St = S[s]
        vn = U[c] - W[c] @ St
        O[c] = scale * (Qg[c] @ St + P[c] @ vn)
        S[s] = el[c] * St + Kd[c] @ vn
    return rows(O, dv), S
