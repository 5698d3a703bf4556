"""Matvecs at the edges of the direct transforms' launch rules: one chunk, whose
M2S goes on to the S2L coefficients (48 particles or fewer), and two or three
(49, 65); partial groups of four particles; one and several right-hand sides.

Tolerances: 1e-11 (FP64, ten times the bound of a single step) and 2e-5 (FP32).
"""
import numpy as np
import pytest

from gpu_common import coeff_vector, gpu_context, make_workload, oracle_problem, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [3, 8, 9, 16])
@pytest.mark.parametrize("n", [1, 15, 48, 49, 65])
def test_chunk_edges(p, n):
    import torch
    wl = make_workload("s70p8", n=n)
    wl.p = p
    wl.n_nodes = 224
    pr = oracle_problem(wl)
    X = np.stack([coeff_vector(wl, 90 + r) for r in range(5)])
    ref = np.stack([pr.matvec(x) for x in X])
    ctx = gpu_context(wl)
    ctx.set_stream(torch.cuda.current_stream().cuda_stream)
    for prec, dt, tol in ((0, np.complex128, 1e-11), (1, np.complex64, 2e-5)):
        assert rel_err(ctx.apply(prec, X[0].astype(dt)), ref[0]) < tol, prec
        xd = torch.from_numpy(X.astype(dt)).cuda()
        yd = torch.full_like(xd, float("nan"))
        ctx.apply_batch_dev(prec, 5, xd, yd)
        torch.cuda.synchronize()
        for r in range(5):
            assert rel_err(yd[r].cpu().numpy(), ref[r]) < tol, (prec, r)
