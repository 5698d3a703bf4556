"""The default M2L form on both sides of its rule's lines (order, particles,
right-hand sides): the vector form for the lowest orders of many pairs, and the
same matvec as every other form.

Tolerances: the parity bounds of the matvec, 1e-11 (FP64) and 2e-5 (FP32).
"""
import numpy as np
import pytest

from gpu_common import coeff_vector, gpu_context, make_workload, rel_err

pytestmark = pytest.mark.gpu

# (precision, order, particles, right-hand sides, form)
SIDES = [(1, 5, 1000, 1, 0), (1, 5, 999, 1, 2), (1, 6, 1000, 1, 2), (1, 1, 1000, 1, 0), (1, 4, 500, 4, 0),
         (1, 4, 499, 4, 2), (0, 3, 2000, 8, 0), (0, 3, 1936, 8, 3), (0, 4, 2000, 8, 3), (0, 1, 1415, 15, 0)]


@pytest.mark.parametrize("prec,p,n,nrhs,form", SIDES)
def test_sides(prec, p, n, nrhs, form):
    import torch
    wl = make_workload("c3", n=n)
    wl.p = p
    x = np.stack([coeff_vector(wl, 30 + r) for r in range(nrhs)])
    xd = torch.from_numpy(x.astype(np.complex64 if prec else np.complex128)).cuda()
    y = {}
    for v in (None, 0, 2, 3):
        ctx = gpu_context(wl)
        if v is not None:
            ctx.set_tuning(prec, v, 0)
        elif nrhs == 1:
            assert ctx.get_tuning(prec)["variant"] == form
        ctx.set_stream(torch.cuda.current_stream().cuda_stream)
        yd = torch.full_like(xd, float("nan"))
        ctx.apply_batch_dev(prec, nrhs, xd, yd)
        torch.cuda.synchronize()
        y[v] = yd.cpu().numpy()
        ctx.close()
    # the rule's form is the one that runs: its sums are the same bits
    assert np.array_equal(y[None], y[form])
    for v in (0, 2, 3):
        assert rel_err(y[None], y[v]) < (2e-5 if prec else 1e-11), v


def test_tuning_of_a_context_without_geometry():
    # the form and the time are known, the chunk count is not: 0 (the rule used to divide by zero)
    import paper_1407_3868_amd as mp
    ctx = mp.Context(0)
    for prec in (0, 1):
        t = ctx.get_tuning(prec)
        assert t["chunks"] == 0 and t["variant"] in (0, 1, 2, 3)
    ctx.set_layers(6.0, 9.0, 12.0, 4.0)
    ctx.set_scattering_matrix(4, 0.3, np.eye(9, dtype=complex))
    assert ctx.get_tuning(0)["chunks"] == 0
    ctx.set_geometry(np.array([[0.0, -2.0]]), np.zeros(1))
    assert ctx.get_tuning(0)["chunks"] == 1 and ctx.get_tuning(1)["chunks"] == 1
