"""The layer forward is no further from the float64 oracle than the plain WY
form (W, U, Q K^T and K^T as the operands of the state pass) evaluated in the
same precision: BOUNDS holds the errors (2-norm of the difference over the
2-norm of the result, exact inverse) that kernels of that form showed on these
inputs on MI355X.  Inputs and kernels are deterministic, so the bounds carry no
margin.

bf16: beta constant and not a bf16 number, keys that share a direction, slow
decay.  An operand that holds beta on its diagonal, rounded, errs by the same
factor in every row, and that adds up over such keys; roundings that differ
from entry to entry do not.  (T diag(beta) as an operand of G and P': 1.11 and
1.16 times the bound on O at C = 64; beta and the unit diagonal outside the
rounded operands: 0.89 and 0.91.)  fp32: drawn and constant beta; the longer
chain of products makes up for its roundings by adding the largest terms last
and the products with the state in two halves (0.54 to 0.90 of the bounds; 1.01
to 1.11 without)."""

import numpy as np
import pytest

from oracle import gdn_forward as fwd

from test_gpu_forward import layer_inputs, run_gpu, stored

pytestmark = pytest.mark.gpu

# (type, beta or None as drawn, share of the common direction, largest decay
# per token): {C: (O, S_final)}
BOUNDS = {
    ("bf16", 0.99, 0.7, 0.01): {16: (5.079e-3, 5.075e-3), 32: (5.728e-3, 5.760e-3),
                                64: (6.585e-3, 7.005e-3)},
    ("bf16", 0.9, 0.9, 0.01): {16: (5.445e-3, 6.256e-3), 32: (6.579e-3, 8.427e-3),
                               64: (8.412e-3, 1.096e-2)},
    ("f32", None, 0.0, 0.01): {16: (3.165e-7, 2.445e-7), 32: (3.213e-7, 2.425e-7),
                               64: (3.330e-7, 2.531e-7)},
    ("f32", 0.9, 0.7, 0.0): {16: (4.873e-7, 4.845e-7), 32: (5.621e-7, 5.845e-7),
                             64: (6.635e-7, 7.078e-7)},
}


def slow_inputs(C, dt, beta, share, decay, L=1024, H=4, d=128):
    """Unit keys with a common direction, log-decays uniform in [-decay, 0]."""
    Q, K, V, b, g, S0 = layer_inputs(C, "f32", B=1, L=L, H=H, seed=C)
    rng = np.random.default_rng(C)
    u = rng.standard_normal((1, 1, H, d))
    K = share * u / np.linalg.norm(u, axis=-1, keepdims=True) + (1 - share ** 2) ** 0.5 * K
    K = K / np.linalg.norm(K, axis=-1, keepdims=True)
    if beta is not None:
        b = np.full_like(b, beta)
    inc = -decay * rng.random((1, L // C, C, H))
    g = np.cumsum(inc, axis=2).reshape(1, L, H).astype(np.float32)
    Q, K, V = (stored(x, dt) for x in (Q, K, V))
    return Q, K, V, b, g, S0


@pytest.mark.parametrize("C", [16, 32, 64])
@pytest.mark.parametrize("case", list(BOUNDS), ids=str)
def test_error_within_that_of_the_wy_form(C, case):
    dt, beta, share, decay = case
    x = slow_inputs(C, dt, beta, share, decay)
    ref = fwd.gdn_chunked(*x[:5], C, x[5], scale=128 ** -0.5)
    got = run_gpu(*x, C, dt, exact=True)
    for a, r, bound, what in zip(got, ref, BOUNDS[case][C], ("O", "S_final")):
        e = float(np.linalg.norm(a - r) / np.linalg.norm(r))
        print(f"C={C} {case} {what}: {e:.4e} (bound {bound:.4e})", flush=True)
        assert e <= bound, what
