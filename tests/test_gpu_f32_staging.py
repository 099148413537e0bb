"""FP32 links staged in LDS or loaded by every lane (the library chooses by the
kind of kernel and the lattice's workgroups): above every line of that choice,
at slice counts with full, ragged and nearly empty wavefronts, all operators
give the same bits either way; and a right-hand side's result in a batch of any
size has the bits it has alone, in the operators and in whole solves."""
import numpy as np
import pytest
import torch

import oracle
from paper_1701_07559_amd import inputs as I

import test_gpu_parity as TP

pytestmark = pytest.mark.gpu
M = TP.M
F32 = 1


def context(M, dims, L5, seed):
    act = oracle.Action(dims, L5, M5=1.3, b5=1.5, c5=0.5, mq=0.05, antiperiodic_t=True)
    return act, TP.make_ctx(M, act, I.random_links(dims, 0.3, seed))


def workgroups(dims, L5):
    per = 4 * (64 // L5)
    return -(-int(np.prod(dims)) // 2 // per)


@pytest.mark.parametrize("dims,L5", [((16, 16, 16, 64), 8), ((16, 16, 16, 58), 9), ((14, 14, 22, 46), 10),
                                     ((14, 18, 18, 38), 12), ((14, 18, 18, 30), 16), ((16, 16, 14, 28), 21),
                                     ((16, 16, 16, 16), 32)], ids=lambda v: str(v) if isinstance(v, int) else "x".join(map(str, v)))
def test_staged_links_give_the_same_bits(M, dims, L5):
    assert workgroups(dims, L5) > 4000
    act, ctx = context(M, dims, L5, 95)
    try:
        base = M.mdwf_get_tune(ctx, F32)
        g = torch.Generator(device="cuda").manual_seed(96)
        x = torch.randn(M.mdwf_field_bytes(ctx, F32, M.MDWF_FULL) // 4, device="cuda", generator=g)
        for op in TP.ALL_OPS:
            out = []
            for lm in (0, 1):
                M.mdwf_set_tune(ctx, F32, dict(base, link_mode=lm))
                o = torch.zeros_like(x)
                torch.cuda.synchronize()
                M.mdwf_apply_dev(ctx, op, F32, x.data_ptr(), o.data_ptr(), stream=torch.cuda.current_stream().cuda_stream)
                torch.cuda.synchronize()
                out.append(o)
            assert bool(torch.isfinite(out[0]).all()) and bool(out[0].any())
            assert torch.equal(out[0], out[1]), "op %d: the link modes differ" % op
    finally:
        M.mdwf_destroy(ctx)


@pytest.mark.parametrize("nrhs", [8, 28])
def test_batch_operator_has_the_bits_of_one(M, nrhs):
    dims, L5 = (8, 8, 8, 16), 9   # 147 workgroups each: 1176 and 4116 together
    act, ctx = context(M, dims, L5, 97)
    assert workgroups(dims, L5) * 8 > 1024 and workgroups(dims, L5) * 28 > 4000
    try:
        fb = M.mdwf_field_bytes(ctx, F32, M.MDWF_FULL)
        g = torch.Generator(device="cuda").manual_seed(98)
        x = torch.randn((nrhs, fb // 4), device="cuda", generator=g)
        st = torch.cuda.current_stream().cuda_stream
        for op in TP.ALL_OPS:
            many, one = torch.zeros_like(x), torch.zeros_like(x)
            torch.cuda.synchronize()
            M.mdwf_apply_batch_dev(ctx, op, F32, nrhs, x.data_ptr(), many.data_ptr(), fb, None, stream=st)
            for k in range(nrhs):
                M.mdwf_apply_dev(ctx, op, F32, x[k].data_ptr(), one[k].data_ptr(), stream=st)
            torch.cuda.synchronize()
            assert bool(one.any()) and torch.equal(many, one), "op %d" % op
    finally:
        M.mdwf_destroy(ctx)


@pytest.mark.parametrize("form", [0, 1, 2])
def test_batch_solve_has_the_bits_of_one(M, form):
    dims, L5 = (8, 8, 8, 16), 9
    act, ctx = context(M, dims, L5, 99)
    bs = [I.gaussian_source(dims, L5, 401 + k) for k in range(8)]
    opts = dict(tol=1e-8, inner=F32, schur_form=form)
    try:
        xs = [np.zeros_like(b) for b in bs]
        st, info = M.mdwf_solve(ctx, bs, xs, opts=opts)
        assert st == M.MDWF_OK
        for k in (0, 3, 7):
            x = np.zeros_like(bs[k])
            st, i1 = M.mdwf_solve(ctx, [bs[k]], [x], opts=opts)
            assert st == M.MDWF_OK and i1[0]["iters"] == info[k]["iters"]
            assert np.array_equal(x, xs[k]), "column %d" % k
    finally:
        M.mdwf_destroy(ctx)
