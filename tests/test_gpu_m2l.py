"""The matrix-core M2L at the edges of its tiles: every kind of order (row
blocks full, partial, with a row on the vector units), one and two target tiles
per wave, ragged targets and source groups, chunks longer than the batches
that the kernels stage, and chunks that hold everything.

Tolerances: the parity bounds of the M2L, 1e-12 (FP64) and 2e-5 (FP32, 300 unit
roundoffs for the growth of the Hankel recurrence); and for FP32 sums over one
long chunk 2e-6 against FP64 (the tables' rounding, 6e-8 times a growth of
about 5, and a sum rounded to nearest: a drifting sum of 1000 sources x 17
orders would show).
"""
import numpy as np
import pytest

from gpu_common import coeff_vector, gpu_context, make_workload, oracle_problem, rel_err
from oracle import operators as oops

pytestmark = pytest.mark.gpu


def _m2l(ctx, prec, x):
    import torch
    xd = torch.from_numpy(x.astype(np.complex128 if prec == 0 else np.complex64)).cuda()
    ad = torch.full_like(xd, float("nan"))
    ctx.set_stream(torch.cuda.current_stream().cuda_stream)
    ctx.m2l_dev(prec, xd, ad)
    torch.cuda.synchronize()
    return ad.cpu().numpy()


@pytest.mark.parametrize("p", [1, 2, 3, 5, 7, 8, 9, 11, 13, 14, 15, 16])
@pytest.mark.parametrize("n", [3, 34, 70])
def test_orders(p, n):
    wl = make_workload("s70p8", n=n)
    wl.p = p
    x = coeff_vector(wl, 50 + p)
    ref = oops.m2l_apply(wl.xy, wl.k2, p, x)
    ctx = gpu_context(wl)
    for prec, tol in ((0, 1e-12), (1, 2e-5)):
        for variant, chunks in ((2, 0), (2, 1), (3, 0), (3, 2)):
            ctx.set_tuning(prec, variant, chunks)
            assert rel_err(_m2l(ctx, prec, x), ref) < tol, (prec, variant, chunks)


@pytest.mark.parametrize("variant", [2, 3])
def test_fp32_long_chunk(variant):
    wl = make_workload("c2")
    wl.p = 8
    x = coeff_vector(wl, 70).astype(np.complex64).astype(np.complex128)
    ctx = gpu_context(wl)
    ref = _m2l(ctx, 0, x)
    ctx.set_tuning(1, variant, 1)
    assert rel_err(_m2l(ctx, 1, x), ref) < 2e-6


@pytest.mark.parametrize("p", [7, 8, 9, 12, 15, 16])
@pytest.mark.parametrize("n,nrhs", [(5, 16), (70, 65), (700, 17)])
def test_many_rhs(p, n, nrhs):
    # one K step (p = 8 .. 15) and the FP32 form beside it; a ragged last group
    # of right-hand sides; chunks longer than the interval between two flushes
    import torch
    wl = make_workload("c2" if n > 70 else "s70p8", n=n)
    wl.p = p
    ctx = gpu_context(wl)
    X = np.stack([coeff_vector(wl, 80 + r) for r in range(3)])[np.arange(nrhs) % 3]
    y = {}
    for prec, dt in ((0, np.complex128), (1, np.complex64)):
        xd = torch.from_numpy(X.astype(dt)).cuda()
        yd = torch.full_like(xd, float("nan"))
        ctx.set_stream(torch.cuda.current_stream().cuda_stream)
        ctx.apply_batch_dev(prec, nrhs, xd, yd)
        torch.cuda.synchronize()
        y[prec] = yd.cpu().numpy()
    assert rel_err(y[0][0], oracle_problem(wl).matvec(X[0])) < 1e-11 if n <= 70 else True
    for r in range(nrhs):
        assert rel_err(y[1][r], y[0][r]) < 2e-5
