"""Device memory that calls take from a context, and calls whose allocation
was refused once: a later call is the one a fresh context makes, bit by bit.
"""
import numpy as np
import pytest

import paper_1407_3868_amd as mp
from gpu_common import coeff_vector, gpu_context, make_workload

pytestmark = pytest.mark.gpu


def _rhs(wl, nrhs, dtype):
    import torch
    x = np.stack([coeff_vector(wl, 90 + r) for r in range(nrhs)]).astype(dtype)
    return torch.from_numpy(x).cuda()


def _batch(ctx, prec, x):
    import torch
    y = torch.full_like(x, float("nan"))
    ctx.set_stream(torch.cuda.current_stream().cuda_stream)
    ctx.apply_batch_dev(prec, x.shape[0], x, y)
    torch.cuda.synchronize()
    return y.cpu().numpy()


@pytest.mark.parametrize("p", [7, 8, 12, 15, 16])
def test_many_rhs_memory(p):
    # beyond what the same call in FP64 holds: the transposed coefficients of
    # whole groups of 64 right-hand sides, rows in fours
    wl = make_workload("s70p8")
    wl.p = p
    ctx = gpu_context(wl)
    x = _rhs(wl, 20, np.complex128)
    _batch(ctx, 0, x)
    before = ctx.memory()[0]
    import torch
    _batch(ctx, 1, x.to(torch.complex64))
    assert ctx.memory()[0] - before <= wl.n * ((wl.P + 3) // 4 * 4) * 64 * 8


def test_refused_call_leaves_no_trace():
    import torch
    wl = make_workload("s70p8")
    wl.p = 12
    x64 = _rhs(wl, 20, np.complex128)
    x = x64.to(torch.complex64)
    ref = _batch(gpu_context(wl), 1, x)
    ctx = gpu_context(wl)
    y64 = torch.empty_like(x64)
    ctx.set_stream(torch.cuda.current_stream().cuda_stream)
    batch = mp.Batch([(ctx, 0, 20, x64, y64)])  # holds the context's buffers
    with pytest.raises(mp.MpslError) as e:
        _batch(ctx, 1, x)
    assert e.value.status == -4
    batch.close()
    assert np.array_equal(_batch(ctx, 1, x), ref)


@pytest.mark.parametrize("p,most", [(1, 9), (8, 9), (11, 9), (12, 17), (16, 17)])
def test_partial_slots_of_large_layouts(p, most):
    # 40000 particles: 2560 blocks of 128 targets, from p = 12 on 10240 of 64
    # (the geometry alone fixes the count; no tables are built)
    ctx = mp.Context(0)
    ctx.set_layers(6.0, 9.0, 12.0, 20.0)
    ctx.set_scattering_matrix(p, 0.3, np.eye(2 * p + 1, dtype=complex))
    i = np.arange(40000)
    ctx.set_geometry(np.stack([0.75 * (i // 20), -1.0 - 0.8 * (i % 20)], 1), np.zeros(i.size))
    for prec in (0, 1):
        assert 1 <= ctx.get_tuning(prec)["chunks"] <= most


@pytest.mark.parametrize("n,p,nr", [(16, 8, 1), (16, 8, 70000), (70, 8, 300), (70, 8, 4096), (203, 16, 4096),
                                    (203, 16, 66000)])
def test_field_at_its_budget(n, p, nr):
    # beyond the tables, the work buffers and one vector (rhs holds one too): receivers,
    # values, three complex numbers per node and layer and the two interfaces
    src = np.array([0.3, 1.5])
    free = _lattice(n, p)
    free.rhs(src)
    need = free.memory()[0] + 2 * nr * 16 + 3 * 3 * 256 * 16 + 2 * 8
    tight = _lattice(n, p, need)
    tight.rhs(src)
    rng = np.random.default_rng(96)
    beta = 1e-3 * (rng.standard_normal((n, 2 * p + 1)) + 1j * rng.standard_normal((n, 2 * p + 1)))
    rcv = np.stack([rng.uniform(-50.0, 50.0, nr), rng.choice([-0.4, -9.2, -12.0, 0.5, 2.0], nr)], 1)
    want = free.eval_field(src, beta, rcv)
    got = tight.eval_field(src, beta, rcv)
    assert np.linalg.norm(got - want) <= 1e-11 * np.linalg.norm(want)
    assert np.array_equal(got, tight.eval_field(src, beta, rcv))


def _lattice(n, p, budget=0, nodes=256, interp=False):
    """n particles (geometry does not change the bytes held), nodes contour nodes."""
    ctx = mp.Context(0, budget)
    ctx.set_layers(6.0, 9.0, 12.0, 10.0)
    ctx.set_scattering_matrix(p, 0.3, 1e-3 * np.eye(2 * p + 1, dtype=complex))
    i = np.arange(n)
    ctx.set_geometry(np.stack([1.8 * (i // 4 - n // 8), -1.5 - 1.8 * (i % 4)], 1), np.zeros(n))
    if interp:
        b, h = mp.span_contour_params(1.8 * n / 4, 1e-6)
        ctx.set_contour_span(b, 24.0, h)
        ctx.set_sommerfeld_method(mp.SOMM_INTERP)
    else:
        ctx.set_contour(nodes, 0.05, 32.0)
    return ctx


def test_matvec_at_its_budget():
    # 203 particles, p = 16, 256 nodes: tables and work buffers of both precisions, and the
    # host calls' staging of two vectors
    need = 20259656 + 2 * 203 * 33 * 16
    free, tight = _lattice(203, 16), _lattice(203, 16, need)
    rng = np.random.default_rng(95)
    for prec, dt in ((0, np.complex128), (1, np.complex64)):
        x = (rng.standard_normal((203, 33)) + 1j * rng.standard_normal((203, 33))).astype(dt)
        assert np.array_equal(tight.apply(prec, x), free.apply(prec, x))


@pytest.mark.parametrize("n,p,most", [(300, 8, 116960836), (300, 16, 158043460)])
def test_interpolated_batch_memory(n, p, most):
    # four right-hand sides over the interpolated transforms: no more than their partials'
    # earlier shape (blocks of four waves) held in all
    import torch
    ctx = _lattice(n, p, interp=True)
    ctx.set_stream(torch.cuda.current_stream().cuda_stream)
    x = torch.zeros(4, n, 2 * p + 1, dtype=torch.complex64, device="cuda")
    ctx.apply_batch_dev(1, 4, x, torch.empty_like(x))
    torch.cuda.synchronize()
    assert ctx.memory()[0] <= most
