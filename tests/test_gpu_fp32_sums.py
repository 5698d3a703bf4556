"""Sums of the FP32 far field: over the partial slots, over the products of the
matrix-core forms, and over the sources of the many-right-hand-side form.

Particles in free space (three equal layers), S = 1: y - x is the summed M2L.
"""
import numpy as np
import pytest

import paper_1407_3868_amd as mp

pytestmark = pytest.mark.gpu


def _context(xy, p):
    import torch
    ctx = mp.Context(0)
    ctx.set_layers(1.0, 1.0, 1.0, 200.0)
    ctx.set_scattering_matrix(p, 0.01, np.eye(2 * p + 1, dtype=complex))
    ctx.set_geometry(xy, np.zeros(len(xy)))
    ctx.set_contour(128, 0.1, 4.0)
    ctx.set_stream(torch.cuda.current_stream().cuda_stream)
    return ctx


def _apply(ctx, prec, x):
    import torch
    y = torch.empty_like(x)
    ctx.apply_batch_dev(prec, x.shape[0], x, y)
    torch.cuda.synchronize()
    return y


def _m2l(ctx, prec, x):
    import torch
    y = torch.empty_like(x)
    ctx.m2l_dev(prec, x, y)
    torch.cuda.synchronize()
    return y


@pytest.mark.parametrize("n", [7, 12, 33, 41])
def test_slots_that_cancel(n):
    # one source per slot; those of coefficients 1 and -1 at the same distance
    # cancel at order 0 of the last particle, and what a third adds stays.  In
    # unit roundoffs: H_0 1, S and the rotation a few; 16 with room.
    import torch
    p, small = 1, 2.0**-13
    a, b, c = (0, 1, 2) if n < 33 else (0, 8, 16)
    xy = np.stack([5.0 + 1.5 * np.arange(n), np.full(n, -100.0)], 1)
    xy[a, 0], xy[b, 0], xy[c, 0], xy[n - 1, 0] = 1.0, 1.5, -1.0, 0.0
    ctx = _context(xy, p)
    ctx.set_tuning(1, 0, n)
    x = np.zeros((n, 2 * p + 1), np.complex128)
    x[a, p], x[b, p], x[c, p] = 1.0, small, -1.0
    x64 = torch.from_numpy(x).cuda()
    x32 = x64.to(torch.complex64)
    ref = complex(_m2l(ctx, 0, x64)[n - 1, p])
    for got in (complex(_m2l(ctx, 1, x32)[n - 1, p]), -complex(_apply(ctx, 1, x32[None])[0, n - 1, p])):
        assert abs(got - ref) <= 16 * 2.0**-24 * abs(ref), (got, ref)


def _error(n, p, call, seeds):
    """Mean over `seeds` of log |FP32 - FP64| / |FP64| of each entry of
    call(ctx, x64, x32) -> (FP64 result, FP32 results), orders weighted."""
    import torch
    w = 0.5 ** np.abs(np.arange(-p, p + 1))
    wt = torch.from_numpy(w).cuda()
    out = []
    for seed in range(seeds):
        rng = np.random.default_rng(300 + seed)
        i = np.arange(n)
        xy = np.stack([3.0 * (i % 40), -20.0 - 3.0 * (i // 40)], 1) + rng.uniform(-0.4, 0.4, (n, 2))
        ctx = _context(xy, p)
        x = (w * (rng.standard_normal((n, 2 * p + 1)) + 1j * rng.standard_normal((n, 2 * p + 1)))).astype(np.complex64)
        x32 = torch.from_numpy(x).cuda()
        ref, got = call(ctx, x32.to(torch.complex128), x32)
        out.append([np.log(float(((g.to(torch.complex128) - ref) * wt).norm() / (ref * wt).norm())) for g in got])
        ctx.close()
    return np.exp(np.mean(out, axis=0))


@pytest.mark.parametrize("p", [4, 8])
def test_matrix_core_sums(p):
    # no further off than the vector form with as many chunks as two sources
    # allow; 700 particles of about six orders that count, 6 seeds: each error
    # to half a percent, 5 % for both
    def call(ctx, x64, x32):
        got = []
        for variant, chunks in ((0, 350), (2, 0), (3, 0)):
            ctx.set_tuning(1, variant, chunks)
            got.append(_m2l(ctx, 1, x32))
        return _m2l(ctx, 0, x64), got

    vector, m16, m32 = _error(700, p, call, 6)
    assert m16 <= 1.05 * vector and m32 <= 1.05 * vector, (m16 / vector, m32 / vector)


@pytest.mark.parametrize("p", [2, 4, 7])
def test_many_rhs_sums(p):
    # sums over at most a fifth of the sources: no further off than the vector
    # form in five chunks (1700 particles, 4 seeds: 5 % for both errors)
    def call(ctx, x64, x32):
        ctx.set_tuning(1, 0, 5)
        one = _apply(ctx, 1, x32[None])[0] - x32
        many = _apply(ctx, 1, x32[None].repeat(16, 1, 1))[3] - x32
        return _apply(ctx, 0, x64[None])[0] - x64, [one, many]

    one, many = _error(1700, p, call, 4)
    assert many <= 1.05 * one, many / one
