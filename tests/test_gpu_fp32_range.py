"""FP32 M2L, for one and for many right-hand sides, over the range of FP32: vectors scaled by powers of two against the
same vectors unscaled, and coefficients next to the largest FP32 number.

Tolerances.  A scaling by 2^-k changes no rounding until products and sums
reach the FP32 subnormals: every sum of a product (six products of parts per
coefficient) may then be off by the smallest of them, 2^-149, so that entries
differ by at most 6 N P 2^(k - 149) after scaling back.  Next to the top of the
range nothing but the usual FP32 rounding applies: 1e-6.
"""
import numpy as np
import pytest

from gpu_common import coeff_vector, gpu_context, make_workload

pytestmark = pytest.mark.gpu


def _apply(ctx, nrhs, x):
    """alpha of one right-hand side, y of several."""
    import torch
    xd = torch.from_numpy(np.ascontiguousarray(x.astype(np.complex64))).cuda()
    yd = torch.full_like(xd, float("nan"))
    ctx.set_stream(torch.cuda.current_stream().cuda_stream)
    if nrhs == 1:
        ctx.m2l_dev(1, xd, yd)
    else:
        ctx.apply_batch_dev(1, nrhs, xd, yd)
    torch.cuda.synchronize()
    return yd.cpu().numpy().astype(np.complex128)


def _workload(p):
    wl = make_workload("s70p8")
    wl.p = p
    return wl


@pytest.mark.parametrize("p", [4, 8, 12, 16])
@pytest.mark.parametrize("variant", [2, 3])
@pytest.mark.parametrize("k", [100, 108, 112, 116, 120])
def test_small_coefficients(p, variant, k):
    wl = _workload(p)
    ctx = gpu_context(wl)
    ctx.set_tuning(1, variant, 0)
    rng = np.random.default_rng(60 + p)
    # coefficients of one size, so that all have the scaled exponent
    x = (rng.uniform(1.0, 2.0, (wl.n, wl.P)) * np.exp(0.25j * np.pi * (1 + 2 * rng.integers(0, 4, (wl.n, wl.P)))))
    x = x.astype(np.complex64).astype(np.complex128)
    ref = _apply(ctx, 1, x)
    got = _apply(ctx, 1, x * 2.0**-k) * 2.0**k
    err = np.linalg.norm(got - ref) / np.sqrt(ref.size)
    assert err <= 6 * wl.n * wl.P * 2.0 ** (k - 149), err


@pytest.mark.parametrize("p,variant", [(4, 2), (8, 2), (4, 3)])
def test_largest_coefficient(p, variant):
    wl = _workload(p)
    ctx = gpu_context(wl)
    ctx.set_tuning(1, variant, 0)
    x = np.zeros((wl.n, wl.P), np.complex128)
    x[7, p] = float(np.finfo(np.float32).max)
    ref = _apply(ctx, 1, x * 2.0**-40) * 2.0**40
    far = np.abs(ref).max(axis=1) < 1e38  # targets whose expansion is far from overflow
    assert far.sum() > wl.n // 2
    got = _apply(ctx, 1, x)
    assert np.isfinite(got[far]).all()
    assert np.linalg.norm((got[far] - ref[far]) / 1e38) <= 1e-6 * np.linalg.norm(ref[far] / 1e38)


@pytest.mark.parametrize("p", [8, 12, 15])
def test_small_coefficients_of_many_rhs(p):
    # each right-hand side alone with its scale: y of several is linear in each;
    # one vector next to the others' size in a group does not lose the others' bits
    wl = _workload(p)
    ctx = gpu_context(wl)
    rng = np.random.default_rng(70 + p)
    x = rng.uniform(1.0, 2.0, (16, wl.n, wl.P)) * np.exp(0.25j * np.pi * (1 + 2 * rng.integers(0, 4, (16, wl.n, wl.P))))
    x = x.astype(np.complex64).astype(np.complex128)
    ref = _apply(ctx, 16, x)
    k = np.array([0, 60, 100, 104, 108, 110, 112, 114, 115, 116, 117, 118, 119, 120, 108, 30])
    scale = 2.0 ** -k[:, None, None]
    got = _apply(ctx, 16, x * scale) / scale
    # a few FP32 roundings that fall the other way, 16 unit roundoffs, and the subnormals'
    # own, independent over the products of the M2L and the terms of the other three steps
    sums = np.sqrt(6 * wl.n * wl.P + 6 * (wl.n * wl.P + 2 * wl.n_nodes))
    for r in range(16):
        rms = np.sqrt(np.mean(np.abs(got[r] - ref[r]) ** 2))
        size = np.sqrt(np.mean(np.abs(ref[r]) ** 2))
        assert rms <= 16 * 2.0**-24 * size + 16 * sums * 2.0 ** (int(k[r]) - 149), (r, int(k[r]), rms / size)
