"""Adjoint launches of small planes, cut into frequency chunks, and their gather with rays
split into groups: the gradient against the oracle's reverse mode, every component, at the
edges of the cut (one frequency; a chunk count that does not divide the frequencies; planes of
less than a wavefront, of ragged blocks, and large enough for the gather's wide blocks and for
one thread per node; ray batches whose last is smaller).  Bars as for the whole adjoint (test_gpu_adjoint_oracle)."""
import numpy as np
import pytest

from paper_1307_4217_amd import inputs, porta
from test_gpu_adjoint_oracle import _compare, _gpu_grad, _oracle_grad, _problem

pytestmark = pytest.mark.gpu

SIZES = [(5, 3, 7, 2, 4, 1), (13, 5, 2, 1, 4, 22), (16, 16, 6, 3, 8, 23), (33, 20, 5, 2, 3, 5),
         (96, 86, 3, 1, 4, 2), (181, 140, 3, 1, 4, 2)]
MODES = [(porta.F64, porta.BILINEAR), (porta.F32, porta.BILINEAR), (porta.F64, porta.BEZIER2D)]


@pytest.mark.parametrize("prec,interp", MODES)
@pytest.mark.parametrize("dims", SIZES)
def test_chunked_adjoint_equals_oracle_gradient(dims, prec, interp):
    cfg = inputs.Config("step", *dims, False)
    freqs = np.arange(cfg.nfreq)
    atm, q, rays, seed, seed_sel = _problem(cfg, prec, freqs, interp)
    ref = _oracle_grad(atm, q, rays, freqs, seed_sel, chunk=25, interp=interp)
    nh = len(q.mu) * q.nchi
    for opts in (None, porta.options(ray_batch=max(1, nh - 1)), porta.options(block=64)):
        got = _gpu_grad(atm, q, prec, seed, stride=min(3, atm.nz - 1), interp=interp, opts=opts)
        _compare(got, ref, prec, str(dims))
