"""Infinities and NaN through every form of the M2L: a coefficient that is not a
finite number reaches every entry of every target, as the sums over all orders
have it, and no other right-hand side.
"""
import numpy as np
import pytest

from gpu_common import coeff_vector, gpu_context, make_workload, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("variant", [0, 2, 3])
@pytest.mark.parametrize("p", [7, 16])
def test_one_right_hand_side(prec, variant, p):
    import torch
    wl = make_workload("s70p8")
    wl.p = p
    ctx = gpu_context(wl)
    ctx.set_tuning(prec, variant, 2)
    ctx.set_stream(torch.cuda.current_stream().cuda_stream)
    for bad in (np.inf, np.nan):
        for m, slot in ((0, 0), (33, p), (69, 2 * p)):
            x = coeff_vector(wl, 51).astype(np.complex64 if prec else np.complex128)
            x[m, slot] = bad
            xd = torch.from_numpy(x).cuda()
            ad = torch.zeros_like(xd)
            ctx.m2l_dev(prec, xd, ad)
            torch.cuda.synchronize()
            assert not np.isfinite(ad.cpu().numpy()).any(), (bad, m, slot)


@pytest.mark.parametrize("p", [7, 12])
def test_many_right_hand_sides(p):
    import torch
    wl = make_workload("s70p8")
    wl.p = p
    ctx = gpu_context(wl)
    ctx.set_stream(torch.cuda.current_stream().cuda_stream)
    x = np.stack([coeff_vector(wl, 52 + r) for r in range(18)]).astype(np.complex64)
    y = {}
    for bad in (0.0, np.inf, np.nan):
        xb = x.copy()
        xb[3, 5, 2] = bad
        xd = torch.from_numpy(xb).cuda()
        yd = torch.zeros_like(xd)
        ctx.apply_batch_dev(1, 18, xd, yd)
        torch.cuda.synchronize()
        y[bad] = yd.cpu().numpy()
    for k in y:
        others = np.arange(18) != 3
        assert np.isfinite(y[k][others]).all()
        assert rel_err(y[k][others], y[0.0][others]) < 2e-5
    assert not np.isfinite(y[np.inf][3]).any() and not np.isfinite(y[np.nan][3]).any()
