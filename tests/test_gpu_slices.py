"""The fifth-dimension recurrences and the staged links of the hop kernels:
every operator at slice counts on both sides of the staging limit (L5 = 8),
with full, nearly empty and ragged wavefronts, term sums up to L5 = 6, for masses 0, 1/20 and 1 and
for actions whose recurrence factor is zero (c5 (4 - M5) = 1: K5 is diagonal;
c5 = 0: B is) or close to one.  Both link modes must give the same bits, and
each operator its oracle value.  The recurrence factors are below one in
modulus for every accepted action, so rounding errors do not grow along it
and the tolerances are those of the other operator tests: a few hundred
units of the last place in FP64, some ten in FP32, the storage in FP16."""
import numpy as np
import pytest

import oracle
from paper_1701_07559_amd import inputs as I

import test_gpu_parity as TP

pytestmark = pytest.mark.gpu
M = TP.M

# dims, L5, (M5, b5, c5, mq)
CASES = [((2, 2, 2, 2), 1, (1.3, 1.5, 0.5, 1.0)), ((4, 2, 2, 2), 2, (1.8, 0.1, 0.0, 0.05)),
         ((2, 4, 2, 2), 3, (1.5, 1.4, 0.4, 0.0)), ((2, 2, 6, 2), 6, (1.8, 0.1, 0.0, 1.0)), ((2, 2, 2, 6), 7, (1.8, 0.1, 0.0, 1.0)),
         ((4, 4, 2, 2), 8, (1.5, 1.4, 0.4, 0.0)), ((2, 2, 2, 2), 8, (1.8, 0.1, 0.0, 1.0)),
         ((2, 4, 4, 2), 9, (1.3, 1.5, 0.5, 1.0)), ((2, 2, 2, 4), 16, (1.8, 0.1, 0.0, 0.0)),
         ((2, 2, 2, 2), 21, (1.5, 1.4, 0.4, 0.05)), ((2, 2, 2, 2), 32, (1.8, 0.1, 0.0, 0.05))]


@pytest.mark.parametrize("prec", [0, 1, 2], ids=lambda p: TP.PREC_NAME[p])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[0])) + "_L%d_m%g" % (c[1], c[2][3]))
def test_recurrences_and_staged_links(M, case, prec):
    dims, L5, (M5, b5, c5, mq) = case
    act = oracle.Action(dims, L5, M5=M5, b5=b5, c5=c5, mq=mq, antiperiodic_t=True)
    U = I.random_links(dims, 0.3, 91)
    psi = I.gaussian_source(dims, L5, 92)
    ctx = TP.make_ctx(M, act, U)
    try:
        base = M.mdwf_get_tune(ctx, prec)
        for op in TP.ALL_OPS:
            ref = TP.oracle_op(M, op, act, U, psi)
            out = []
            for lm in (0, 1):
                M.mdwf_set_tune(ctx, prec, dict(base, link_mode=lm))
                out.append(TP.gpu_op(M, ctx, op, prec, act, psi))
            err = TP.rel(out[0], ref)
            assert err <= TP.TOL[prec], "op %d: rel err %.3e" % (op, err)
            assert np.array_equal(out[0], out[1]), "op %d: the link modes differ" % op
    finally:
        M.mdwf_destroy(ctx)


@pytest.mark.parametrize("dims", [(16, 16, 16, 14), (16, 16, 16, 18)], ids=["896wg", "1152wg"])
def test_staged_links_by_launch_size(M, dims):
    """FP32 launches stage the links from 1025 workgroups on: on both sides of
    that the operators give the bits of link mode 0."""
    L5 = 8
    act = oracle.Action(dims, L5, M5=1.3, b5=1.5, c5=0.5, mq=0.05, antiperiodic_t=True)
    ctx = TP.make_ctx(M, act, I.random_links(dims, 0.3, 93))
    rng = np.random.default_rng(94)
    vh = int(np.prod(dims)) // 2
    psi = rng.normal(size=(L5, vh, 4, 3)) + 1j * rng.normal(size=(L5, vh, 4, 3))
    try:
        base = M.mdwf_get_tune(ctx, 1)
        for op in (M.MDWF_OP_HOP_EO, M.MDWF_OP_SCHUR, M.MDWF_OP_SCHUR_DAG, M.MDWF_OP_SCHUR_RP, M.MDWF_OP_SCHUR_RP_DAG):
            out = []
            for lm in (0, 1):
                M.mdwf_set_tune(ctx, 1, dict(base, link_mode=lm))
                o = np.zeros_like(psi)
                M.mdwf_apply(ctx, op, 1, psi, o)
                out.append(o)
            assert np.isfinite(out[0]).all() and np.array_equal(out[0], out[1]), "op %d" % op
    finally:
        M.mdwf_destroy(ctx)
