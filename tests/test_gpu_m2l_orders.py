"""The highest orders of the FP64 M2L: one source coefficient of order +-p meets
h_{+-2p} at the targets' orders -+p, on a line, where e^{iq phi} is +-1.

Tolerance for p = 16, root mean square over the targets, in unit roundoffs:
2/z is rounded once (0.41) and enters 31 times, 13; 31 rounded multiples and
multiply-adds, 0.41 each and independent, 3; H_0 and H_1 up to 3 each, 6; all
together 24 with the reference's own.
"""
import numpy as np
import pytest
import scipy.special as sp

import paper_1407_3868_amd as mp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", [0, 2, 3])
def test_recurrence(variant):
    import torch
    p, n = 16, 201
    rng = np.random.default_rng(17)
    x = np.concatenate([[0.0], 2.0 + 0.06 * np.arange(n - 1) + rng.uniform(0.0, 0.03, n - 1)])
    ctx = mp.Context(0)
    ctx.set_layers(1.0, 1.0, 1.0, 4.0)
    ctx.set_scattering_matrix(p, 0.01, np.eye(2 * p + 1, dtype=complex))
    ctx.set_geometry(np.stack([x, np.full(n, -2.0)], 1), np.zeros(n))
    ctx.set_contour(128, 0.1, 4.0)
    ctx.set_tuning(0, variant, 0)
    ctx.set_stream(torch.cuda.current_stream().cuda_stream)
    z = x[1:].astype(np.longdouble)
    h = [sp.j0(x[1:]) + 1j * sp.y0(x[1:]).astype(np.clongdouble), sp.j1(x[1:]) + 1j * sp.y1(x[1:]).astype(np.clongdouble)]
    for q in range(2, 2 * p + 1):
        h.append(2 * (q - 1) / z * h[-1] - h[-2])
    for sign in (1, -1):  # h_q = H_q e^{iq phi}, phi = 0; h_{-q} = (-1)^q H_q
        beta = np.zeros((n, 2 * p + 1), np.complex128)
        beta[0, p + sign * p] = 1.0
        b = torch.from_numpy(beta).cuda()
        a = torch.empty_like(b)
        ctx.m2l_dev(0, b, a)
        torch.cuda.synchronize()
        got = a.cpu().numpy()[1:, p - sign * p]
        err = np.abs((got - h[2 * p]) / h[2 * p])
        rms = float(np.sqrt(np.mean(err**2))) / 2.0**-53
        assert rms <= 24, rms
