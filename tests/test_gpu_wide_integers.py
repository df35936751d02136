"""Backward products whose gradient's integers are far wider than the operands' (marked gpu): a
grad plan with t_bits far below p, against exact integer arithmetic."""
import numpy as np
import pytest

import synth
from tests.gpu_util import dev_mp, mp_to_ints, need_gpu

pytestmark = pytest.mark.gpu


def _round(x, p):
    """(sign, significand, exponent) of x 2^0 rounded to p bits, nearest-even, value sign * s * 2^(e - p)."""
    if x == 0:
        return 0, 0, 0
    s, a = (1 if x > 0 else -1), abs(x)
    sh = a.bit_length() - p
    if sh > 0:
        q, r = a >> sh, a & ((1 << sh) - 1)
        q += r > 1 << (sh - 1) or (r == 1 << (sh - 1) and q & 1)
    else:
        q = a << -sh
    e = sh + p
    return (s, q, e) if q >> p == 0 else (s, q >> 1, e + 1)


# 121, 124, 125, 126 and 204 words of the gradient: pairs of moduli up to 124 digits, single ones above
@pytest.mark.parametrize("p", [3840, 3945, 3960, 4000, 6500])
def test_gradient_wider_than_the_operands(p):
    need_gpu()
    from paper_2609_27831_amd import oz2h as oz
    M, N, K = 3, 5, 4
    nl = (p + 63) // 64
    A, B, W = (synth.mp_random(p + i, *s, p, 0, 0) for i, s in enumerate([(M, K), (K, N), (M, N)]))
    for X in (A, B):   # short operands: exact at 100 bits
        X.limbs[..., :nl - 1] = 0
    plan = oz.Plan.create_grad(p, M, N, K, oz.default_opts(t_bits=100))
    print(f"p = {p}: {plan.nw32} words", flush=True)
    ws = oz.workspace(plan, M, N)
    oz.gemm(plan, dev_mp(A), dev_mp(B), ws=ws)
    a, b, w = (np.array(mp_to_ints(X.sign, X.limbs), dtype=object).reshape(X.sign.shape) for X in (A, B, W))
    for got, want in zip(oz.gemm_backward(plan, ws, dev_mp(W)), (w.dot(b.T), a.T.dot(w))):
        s, e, l = got.to_host()
        ints = mp_to_ints(s, l)
        for (i, x), g, ee in zip(np.ndenumerate(want), ints, e.reshape(-1)):
            sx, qx, ex = _round(x, p)
            assert (g, int(ee)) == (sx * qx, ex - 2 * p), i
