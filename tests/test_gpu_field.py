"""Field evaluation against the oracle at the edges of its launch shape: one
receiver, the counts around a block of 256, receivers in every layer, several
chunks of particles and of nodes, particles near enough for the library Bessel
functions and far enough for the expansion, and the small-scratch path of a
context at its memory budget.

Tolerance: relative 2-norm 1e-11, the per-entry bound of the FP64 steps (sums
of at most N P + 2 N_S terms of a few ulp each).
"""
import numpy as np
import pytest

import paper_1407_3868_amd as mp
from gpu_common import coeff_vector, gpu_context, make_workload, oracle_problem, prototype_S, rel_err
from synth.layouts import receivers

pytestmark = pytest.mark.gpu

TOL = 1e-11


def _receivers(wl, count, seed):
    x = wl.xy[:, 0]
    return receivers(count, (x.min() - 2.0, x.max() + 2.0), (-wl.d - 2.0, 3.0), wl.xy, seed, wl.r_enclose + 0.05,
                     wl.src[0])


@pytest.mark.parametrize("name,count", [("c1", 1), ("c1", 63), ("s70p8", 255), ("s150p12", 257), ("s200p16", 1000)])
def test_field_counts(name, count):
    wl = make_workload(name)
    beta = coeff_vector(wl, 41)
    rcv = _receivers(wl, count, 43)
    got = gpu_context(wl).eval_field(wl.src[0], beta, rcv)
    ref = oracle_problem(wl).field(wl.src[0], beta, rcv)
    assert rel_err(got, ref) < TOL, rel_err(got, ref)


def test_field_small_scratch():
    wl = make_workload("s70p8")
    beta = coeff_vector(wl, 44)
    rcv = _receivers(wl, 700, 45)
    ctx = gpu_context(wl)
    ctx.rhs(wl.src[0])
    used = ctx.memory()[0]
    full = ctx.eval_field(wl.src[0], beta, rcv)
    # room for the staging and for two slots of 256 receivers, not for every chunk of 700
    need = beta.size * 16 + 2 * 700 * 16 + 16 * (9 * wl.n_nodes + 2 * 256) + 8 * 12
    tight = mp.Context(0, used + need + 1024)
    tight.set_layers(wl.k1, wl.k2, wl.k3, wl.d)
    tight.set_scattering_matrix(wl.p, wl.r_enclose, prototype_S(wl))
    tight.set_geometry(wl.xy, wl.rot)
    tight.set_contour(wl.n_nodes, wl.b, wl.t_max)
    tight.rhs(wl.src[0])
    got = tight.eval_field(wl.src[0], beta, rcv)
    assert rel_err(got, full) < TOL, rel_err(got, full)


def test_field_inside():
    wl = make_workload("s70p8")
    beta = coeff_vector(wl, 46)
    rcv = np.concatenate([_receivers(wl, 300, 47), wl.xy[-1:] + [0.5 * wl.r_enclose, 0.0], wl.xy[:1]])
    u = gpu_context(wl).eval_field(wl.src[0], beta, rcv)
    assert np.isfinite(u[:300]).all() and np.isnan(u[300:].real).all()
