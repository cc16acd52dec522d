"""The integer inverses form their sums in narrow arithmetic (fp32 at 8 bits;
int32 rounded to odd at 16 bits) where the terms' exponents allow it and in
fp64 elsewhere.  Tiles whose amplitude, density and exponent vary widely put
the exponent gaps of every Add and of the two three-term sums on both sides
of each limit (products below 2^23, gaps of 14 and more, terms finer than the
rounding unit), and the codes and exponents must still equal the exact
integer oracle's, in both forms."""

import numpy as np
import pytest
import torch

from oracle import int8 as oi

import paper_2606_06034_amd as G

pytestmark = pytest.mark.gpu


def graded_tiles(n, C, qmax, seed):
    """Strictly lower codes: amplitude 2^k, k drawn per tile up to the code
    range, entries kept with a density drawn per tile, the far sub-diagonals
    damped in half of the tiles; exponents in the convergent range (every row
    of |A| sums below 1)."""
    rng = np.random.default_rng([seed, C, qmax])
    bits = int(np.log2(qmax + 1))
    q = np.zeros((n, C, C), np.int64)
    e = np.zeros(n, np.int64)
    i, j = np.tril_indices(C, -1)
    for t in range(n):
        amp = min(qmax, 2 ** int(rng.integers(1, bits + 1)))
        v = rng.integers(-amp, amp + 1, size=i.size)
        v = np.where(rng.random(i.size) < rng.choice([0.03, 0.2, 1.0]), v, 0)
        if t % 2:
            v = np.trunc(v * 0.5 ** ((i - j - 1) / rng.uniform(1.0, 8.0))).astype(np.int64)
        q[t, i, j] = v
        top = -(int(np.ceil(np.log2(amp + 1))) + int(np.log2(C)))
        e[t] = top - int(rng.choice([0, 1, 3, 7, 12, 17, 25]))
    return q, e


@pytest.mark.parametrize("plain", [False, True])
@pytest.mark.parametrize("C,N,S", [(16, 3, 2), (32, 3, 4), (64, 3, 8), (64, 1, 5), (32, 0, 3)])
@pytest.mark.parametrize("width", [8, 16])
def test_graded_tiles_bit_exact(width, C, N, S, plain):
    qmax = 127 if width == 8 else 32639
    q, e = graded_tiles(48, C, qmax, seed=width + N + S)
    print(f"graded int{width} C={C} N={N} S={S} plain={plain}", flush=True)
    dt = torch.int8 if width == 8 else torch.int16
    f = G.gdn_chunk_inverse_neumann_i8 if width == 8 else G.gdn_chunk_inverse_neumann_i16
    ref = oi.neumann_inverse_int8 if width == 8 else oi.neumann_inverse_int16
    Tq, eT = f(torch.from_numpy(q).to(dt).cuda(), torch.from_numpy(e).to(torch.int32).cuda(), N, S,
               plain=plain)
    rq, re, _ = ref(q, e, N, S, plain=plain)
    assert np.array_equal(Tq.cpu().numpy().astype(np.int64), rq)
    assert np.array_equal(eT.cpu().numpy().astype(np.int64), re)
