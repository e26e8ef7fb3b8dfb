"""Columns so long, with so many rays, that a call holds the rays' geometry for a window of layers
at a time (porta_abi.hip: kGeomBytes; less in the static scratch of the no-alloc call): 2048 rays
a hemisphere on 2099 layers, whose window of 2048 layers moves once, about 500 in the scratch, and
a ray batch that leaves a smaller last one.  Against the oracle in FP64, at the bars of the sweep
and of the adjoint, and in either precision against calls that hold the whole table."""
import dataclasses

import numpy as np
import pytest

from gpu_common import Case, compare_jkq, compare_stokes, rounded, up_rays
from paper_1307_4217_amd import inputs, porta
from test_gpu_adjoint_oracle import _compare, _gpu_grad, _oracle_grad, _problem

pytestmark = pytest.mark.gpu

CFG = inputs.Config("column", 1, 1, 2100, 64, 32, 1, True)


def _sweeps(case, atm):
    """Whole batches, batches whose last is smaller, the static scratch."""
    import torch
    got = [case.sweep(), case.sweep(opts=porta.options(ray_batch=1500))]
    jkq = torch.empty((10, case.hg.N), dtype=torch.float64, device="cuda")
    itop = torch.empty((2048, 1, 1, 1, 4), dtype=case.dt, device="cuda")
    porta.fs_sweep_noalloc(case.hg, case.kappa, case.prop, case.emis, atm.i_bottom, jkq, itop,
                           atm.w2, prec=case.prec)
    torch.cuda.synchronize()
    return got + [(jkq.cpu().numpy(), itop.cpu().numpy())]


def test_sweeps_in_windows_of_layers_match_oracle(orc):
    atm = inputs.make_atmosphere(CFG, seed=8)
    q = inputs.make_quadrature(CFG)
    ref = orc.fs_sweep(orc.OracleProblem(atm, q))
    print("oracle done", flush=True)
    for j, it in _sweeps(Case(atm, q, porta.F64), atm):
        compare_stokes(it, up_rays(ref["itop"], q), 1e-10, 1e-12, "column")
        compare_jkq(j, ref["jkq"], 1e-10, "column")


@pytest.mark.parametrize("prec", [porta.F64, porta.F32])
def test_sweeps_in_windows_of_layers_equal_those_without(prec):
    """The rays of one inclination in a quadrature of their own, whose geometry is held whole: the
    same Stokes vectors bit for bit."""
    atm = inputs.make_atmosphere(CFG, seed=8)
    if prec == porta.F32:
        atm = rounded(atm, np.float32)
    q = inputs.make_quadrature(CFG)
    got = _sweeps(Case(atm, q, prec), atm)
    for a in (0, 31, 63):
        one = dataclasses.replace(q, mu=q.mu[a:a + 1], wmu=np.ones(1))
        _, want = Case(atm, one, prec).sweep()
        for _, it in got:
            np.testing.assert_array_equal(it[32 * a:32 * (a + 1)], want)


def test_adjoint_in_windows_of_layers_matches_oracle():
    freqs = np.arange(1)
    atm, q, rays, seed, seed_sel = _problem(CFG, porta.F64, freqs)
    ref = _oracle_grad(atm, q, rays, freqs, seed_sel)
    for opts in (None, porta.options(ray_batch=2047)):
        got = _gpu_grad(atm, q, porta.F64, seed, stride=40, opts=opts)
        _compare(got, ref, porta.F64, "column")
