"""9-point adjoints of large planes and few rays, whose gather takes a node and a group of
components a thread.  FP64 against the oracle's reverse mode at the bars of the whole adjoint: one
ray whose frequencies are in several chunks, last blocks of a few nodes and the smallest plane of
the rule.  Larger planes, where elements of 1e-6 of the largest carry 1e-8 of conditioning, and
FP32, which the kinks of the limited interpolation keep from such a comparison, against the
calls that gather all rays at once, a component a thread: both add the same values in FP64, but
for chunks of frequencies (a rounding of 6e-8 a value in FP32, sums of up to ten times the
result: 1e-6 of each field's largest; in FP64 1e-13, as between cuts elsewhere)."""
import numpy as np
import pytest

from gpu_common import rounded
from paper_1307_4217_amd import inputs, porta
from test_gpu_adjoint_oracle import _compare, _gpu_grad, _oracle_grad, _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(128, 129, 3, 1, 1, 4), (3, 5462, 3, 1, 1, 3),
                                  (128, 128, 4, 1, 2, 2)])
def test_few_ray_gather_equals_oracle_gradient(dims):
    cfg = inputs.Config("bez", *dims, False)
    freqs = np.arange(cfg.nfreq)
    atm, q, rays, seed, seed_sel = _problem(cfg, porta.F64, freqs, porta.BEZIER2D)
    ref = _oracle_grad(atm, q, rays, freqs, seed_sel, chunk=25, interp=porta.BEZIER2D)
    got = _gpu_grad(atm, q, porta.F64, seed, stride=2, interp=porta.BEZIER2D)
    _compare(got, ref, porta.F64, str(dims))


@pytest.mark.parametrize("prec,dims,batches", [(porta.F32, (128, 129, 3, 1, 5, 3), (1, 2)),
                                               (porta.F32, (193, 192, 3, 1, 6, 2), (1, 2, 4)),
                                               (porta.F64, (193, 192, 3, 1, 13, 2), (2, 5, 12))])
def test_few_ray_gather_equals_all_rays_at_once(prec, dims, batches):
    cfg = inputs.Config("bez", *dims, False)
    atm = rounded(inputs.make_atmosphere(cfg, seed=4), np.float32)
    q = inputs.make_quadrature(cfg)
    nh = len(q.mu) * q.nchi
    seed = np.random.default_rng(3).standard_normal((nh, cfg.nfreq, cfg.ny, cfg.nx, 4))
    bar = 1e-13 if prec == porta.F64 else 1e-6
    ref = _gpu_grad(atm, q, prec, seed, stride=2, interp=porta.BEZIER2D)
    for batch in batches:
        got = _gpu_grad(atm, q, prec, seed, stride=2, interp=porta.BEZIER2D,
                        opts=porta.options(ray_batch=batch))
        for a, b in zip(got, ref):
            assert np.abs(a - b).max() <= bar * np.abs(b).max(), (prec, dims, batch)
