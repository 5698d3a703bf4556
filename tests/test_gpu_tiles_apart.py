"""Interpolated transforms over tiles that stand apart (no neighbours to share an
exponential with) on both sides of the rule that then drops the padding: 15 and
16 lone tiles, a last step that is not full, pairs among lone tiles, and two rows.

Tolerances as in the tests of uneven tiles: 1e-10 (FP64) and 2e-5 (FP32).
"""
import numpy as np
import pytest

import paper_1407_3868_amd as mp
from gpu_common import make_workload, rel_err
from oracle import contour as ocontour
from oracle import operators as oops

pytestmark = pytest.mark.gpu


def _xy(name, d):
    c = {"lone15": 5 * np.arange(15), "lone16": 5 * np.arange(16), "lone37": 6 * np.arange(37),
         "pairs": np.concatenate([5 * np.arange(24), 5 * np.arange(3) + 1]), "rows": 5 * np.arange(20)}[name]
    xy = np.stack([8.0 * c + 0.5 + np.arange(c.size) % 5, -d + 1.3 + 0.1 * (np.arange(c.size) % 7)], axis=1)
    if name == "rows":
        xy[::3, 1] += 4.0
    xy = np.concatenate([xy, xy[:4] + [1.5, 0.9]])  # a few tiles with two
    return np.ascontiguousarray(xy)


@pytest.mark.parametrize("name", ["lone15", "lone16", "lone37", "pairs", "rows"])
def test_tiles_apart(name):
    import torch
    wl = make_workload("s150p12")
    p, d = 8, 12.0
    xy = _xy(name, d)
    n, P = len(xy), 2 * p + 1
    lam, w = ocontour.contour_span(0.01, 24.0, 0.03, [wl.k1, wl.k2, wl.k3])
    rng = np.random.default_rng(6)
    x = rng.standard_normal((n, P)) + 1j * rng.standard_normal((n, P))
    sig = rng.standard_normal((2, lam.size)) + 1j * rng.standard_normal((2, lam.size))
    ctx = mp.Context(0)
    ctx.set_sommerfeld_method(mp.SOMM_INTERP)
    ctx.set_layers(wl.k1, wl.k2, wl.k3, d)
    ctx.set_scattering_matrix(p, 0.2, np.eye(P, dtype=np.complex128))
    ctx.set_geometry(xy, np.zeros(n))
    ctx.set_contour_span(0.01, 24.0, 0.03)
    ctx.set_stream(torch.cuda.current_stream().cuda_stream)
    m2s = np.stack(oops.m2s(x, xy, lam, wl.k2, d))
    s2l = oops.s2l(sig[0], sig[1], xy, lam, w, wl.k2, d, p)
    for prec, dt, tol in ((0, np.complex128, 1e-10), (1, np.complex64, 2e-5)):
        sd = torch.full((2, lam.size), float("nan"), dtype=torch.complex128, device="cuda")
        ctx.m2s_dev(prec, torch.from_numpy(x.astype(dt)).cuda(), sd)
        ad = torch.full((n, P), float("nan"), dtype=torch.complex128 if prec == 0 else torch.complex64, device="cuda")
        ctx.s2l_dev(prec, torch.from_numpy(sig).cuda(), ad)
        torch.cuda.synchronize()
        assert rel_err(sd.cpu().numpy(), m2s) < tol, prec
        assert rel_err(ad.cpu().numpy(), s2l) < tol, prec


@pytest.mark.parametrize("step", [1, 2, 4])
def test_fp32_error_over_gaps(step):
    # M2S in FP32 against FP64, tiles `step` widths apart.  Per tile and node two FP32
    # exponentials (reduced argument, series, exp of the real part, product: 1.7 unit roundoffs
    # root mean square each), the tile's sum and the product with it, 1 each: 3.5 with a
    # quarter to spare; nothing more for the steps from tile to tile
    import torch
    wl = make_workload("s150p12")
    p, d, n = 8, 12.0, 64
    i = np.arange(n)
    xy = np.stack([8.0 * step * i + 0.5, -0.5 * d + 0.3 * np.sin(i)], axis=1)
    rng = np.random.default_rng(8)
    ctx = mp.Context(0)
    ctx.set_sommerfeld_method(mp.SOMM_INTERP)
    ctx.set_layers(wl.k1, wl.k2, wl.k3, d)
    ctx.set_scattering_matrix(p, 0.2, np.eye(2 * p + 1, dtype=np.complex128))
    ctx.set_geometry(xy, np.zeros(n))
    ctx.set_contour(4096, 1e-3, 32.0)
    ctx.set_stream(torch.cuda.current_stream().cuda_stream)
    decay = 0.3 ** np.abs(np.arange(-p, p + 1))
    x = (rng.standard_normal((n, 2 * p + 1)) + 1j * rng.standard_normal((n, 2 * p + 1))) * decay
    x = torch.from_numpy(x.astype(np.complex64)).cuda()
    s64 = torch.zeros(2, 4096, dtype=torch.complex128, device="cuda")
    s32 = torch.zeros_like(s64)
    ctx.m2s_dev(0, x.to(torch.complex128), s64)
    ctx.m2s_dev(1, x, s32)
    torch.cuda.synchronize()
    err = rel_err(s32.cpu().numpy(), s64.cpu().numpy())
    assert err <= 3.5 * 2.0**-24, err
