"""Coefficients of the hop kernels' fifth-dimension operators in FP32: with all
links zero, S B^-1 is its centre term K5 B^-1, so a field that is 1 on one slice
and 0 on the others returns one coefficient of it per slice.  Every coefficient
is formed in more than FP32 and rounded once, so each entry is the exact value
(rational arithmetic on the action's parameters) to half a unit of the last
place, for the term sums (L5 <= 6) and the recurrences (L5 >= 7), up to factors
c5 / b5 close to one."""
from fractions import Fraction as F

import numpy as np
import pytest

import oracle

import test_gpu_parity as TP

pytestmark = pytest.mark.gpu
M = TP.M

ACTIONS = [(1.3, 1.5, 0.5), (1.5, 1.5, 1.4), (1.9, 1.0, 0.95), (1.8, 0.1, 0.0)]


def coefficients(M5, b5, c5, mq, L5):
    """K5 B^-1 = sum_k c[k] C^k with C^L5 = -m_q."""
    M5, b5, c5, mq = (F(float(v)) for v in (M5, b5, c5, mq))
    ka, kb, z = 1 + b5 * (4 - M5), c5 * (4 - M5) - 1, -c5 / b5
    inv = [z ** k / (b5 * (1 + mq * z ** L5)) for k in range(L5)]   # B^-1
    return [ka * inv[k] + (kb * inv[k - 1] if k else -mq * kb * inv[L5 - 1]) for k in range(L5)], mq


@pytest.mark.parametrize("L5", [1, 2, 4, 5, 6, 7, 8, 13, 21])
@pytest.mark.parametrize("action", ACTIONS, ids=lambda a: "M%g_b%g_c%g" % a)
def test_impulse_response(M, action, L5):
    dims, mq = (2, 2, 2, 2), 0.3
    act = oracle.Action(dims, L5, *action, mq=mq)
    coef, mq = coefficients(*action, mq, L5)
    ctx = TP.make_ctx(M, act, np.zeros((2, 2, 2, 2, 4, 3, 3), complex))
    # half a unit of the last place, and the FP64 sums' own rounding beside it
    tol = 2.0 ** -24 * (1 + 1e-6)
    try:
        for op, adj in ((M.MDWF_OP_SCHUR_RP, False), (M.MDWF_OP_SCHUR_RP_DAG, True)):
            for s0 in range(L5):
                x = np.zeros((L5, 8, 4, 3), complex)
                x[s0] = 1.0
                out = np.zeros_like(x)
                M.mdwf_apply(ctx, op, M.MDWF_F32, x, out)
                for half in (0, 1):   # C moves the upper spins up, the lower down; its adjoint the other way
                    got = out[:, :, 2 * half: 2 * half + 2].reshape(L5, -1)
                    up = (half == 0) != adj
                    for s in range(L5):
                        k = (s - s0 if up else s0 - s) % L5
                        wall = (s < s0) if up else (s > s0)
                        ref = float(coef[k] * (-mq if wall else 1))
                        assert np.all(got[s] == got[s, 0]) and got[s, 0].imag == 0.0
                        assert abs(got[s, 0].real - ref) <= tol * abs(ref), \
                            "op %d slice %d from %d: %.9g, exact %.9g" % (op, s, s0, got[s, 0].real, ref)
    finally:
        M.mdwf_destroy(ctx)
