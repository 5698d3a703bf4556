"""Interpolated transforms over uneven tiles: rows of tiles with gaps that end
a group of four neighbours and gaps that do not, single tiles, tiles with more
than 16 particles, and a last group that is not full.

Tolerances: those of the interpolated transforms, 1e-10 (FP64, interpolation
error about 1e-13) and 2e-5 (FP32).
"""
import numpy as np
import pytest

import paper_1407_3868_amd as mp
from gpu_common import make_workload, prototype_S, rel_err
from oracle import contour as ocontour
from oracle import operators as oops

pytestmark = pytest.mark.gpu

# (column, row, particles) of tiles 8 wide and 4 high: steps of 1, 2, 4 (kept in
# a group), 5 and 9 (a new group), a run of six, a lone tile
TILES = {
    "gaps": [(0, 0, 1), (1, 0, 20), (3, 0, 3), (7, 0, 2), (12, 0, 1), (21, 0, 4), (2, 1, 5)],
    "runs": [(c, 0, 1 + c % 3) for c in range(6)] + [(c, 1, 17 if c == 9 else 2) for c in range(4, 13)],
    "one": [(0, 0, 3)],
}


def _geometry(wl, tiles):
    # 24 sites of 1.25 x 0.9 in a tile; the first particle of the first tile
    # fixes the grid's origin
    pts = []
    for c, r, k in tiles:
        s = np.arange(k)
        pts.append(np.stack([8.0 * c + 0.1 + 1.25 * (s % 6), -wl.d + 1.0 + 4.0 * r + 0.1 + 0.9 * (s // 6)], axis=1))
    xy = np.concatenate(pts)
    assert xy[:, 1].max() < -0.5
    return np.ascontiguousarray(xy[np.random.default_rng(5).permutation(len(xy))])


@pytest.mark.parametrize("p", [8, 9])
@pytest.mark.parametrize("name", list(TILES))
def test_uneven_tiles(name, p):
    import torch
    wl = make_workload("s150p12")
    wl.p = p
    wl.d = 12.0
    xy = _geometry(wl, TILES[name])
    n, P = len(xy), 2 * p + 1
    lam, w = ocontour.contour_span(0.02, 24.0, 0.03, [wl.k1, wl.k2, wl.k3])
    rng = np.random.default_rng(6)
    x = rng.standard_normal((n, P)) + 1j * rng.standard_normal((n, P))
    sig = rng.standard_normal((2, lam.size)) + 1j * rng.standard_normal((2, lam.size))
    ctx = mp.Context(0)
    ctx.set_sommerfeld_method(mp.SOMM_INTERP)
    ctx.set_layers(wl.k1, wl.k2, wl.k3, wl.d)
    ctx.set_scattering_matrix(p, 0.2, np.eye(P, dtype=np.complex128))
    ctx.set_geometry(xy, np.zeros(n))
    ctx.set_contour_span(0.02, 24.0, 0.03)
    ctx.set_stream(torch.cuda.current_stream().cuda_stream)
    m2s = np.stack(oops.m2s(x, xy, lam, wl.k2, wl.d))
    s2l = oops.s2l(sig[0], sig[1], xy, lam, w, wl.k2, wl.d, p)
    for prec, dt, tol in ((0, np.complex128, 1e-10), (1, np.complex64, 2e-5)):
        sd = torch.full((2, lam.size), float("nan"), dtype=torch.complex128, device="cuda")
        ctx.m2s_dev(prec, torch.from_numpy(x.astype(dt)).cuda(), sd)
        ad = torch.full((n, P), float("nan"), dtype=torch.complex128 if prec == 0 else torch.complex64, device="cuda")
        ctx.s2l_dev(prec, torch.from_numpy(sig).cuda(), ad)
        torch.cuda.synchronize()
        assert rel_err(sd.cpu().numpy(), m2s) < tol, prec
        assert rel_err(ad.cpu().numpy(), s2l) < tol, prec
