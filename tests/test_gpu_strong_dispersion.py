"""Sweep and gradient where the dispersion exceeds the absorption by up to 30 (strong Faraday
rotation) against the oracle: the solve's terms of size rho^2 must not cancel.  Bars as for the
whole sweep and adjoint."""
import dataclasses

import numpy as np
import pytest

import test_gpu_adjoint_oracle as adj
from gpu_common import Case, compare_jkq, compare_stokes, rounded, up_rays
from paper_1307_4217_amd import inputs, porta

pytestmark = pytest.mark.gpu

CFG = inputs.Config("dispersion", 12, 10, 9, 2, 4, 7, True)


@pytest.fixture
def strong(monkeypatch):
    """make_atmosphere with rho of 20 to 30 eta_I in random directions."""
    plain = inputs.make_atmosphere

    def make(cfg, seed=0, **kw):
        atm = plain(cfg, seed=seed, **kw)
        rng = np.random.default_rng(99)
        d = rng.normal(size=(3, atm.npoints))
        d *= rng.uniform(20, 30, atm.npoints) / np.linalg.norm(d, axis=0)
        prop = atm.propmat.copy()
        prop[3:] = d * atm.kappa
        return dataclasses.replace(atm, propmat=prop)

    monkeypatch.setattr(inputs, "make_atmosphere", make)


@pytest.mark.parametrize("prec", [porta.F64, porta.F32])
def test_sweep_matches_oracle(orc, strong, prec):
    atm = inputs.make_atmosphere(CFG, seed=1)
    if prec == porta.F32:
        atm = rounded(atm, np.float32)
    q = inputs.make_quadrature(CFG)
    assert (np.linalg.norm(atm.propmat[3:], axis=0) / atm.kappa).min() > 19
    ref = orc.fs_sweep(orc.OracleProblem(atm, q))
    jkq, itop = Case(atm, q, prec).sweep()
    tol_i, tol_p = (1e-10, 1e-12) if prec == porta.F64 else (2e-5, 1e-7)
    compare_stokes(itop, up_rays(ref["itop"], q), tol_i, tol_p, "dispersion")
    compare_jkq(jkq, ref["jkq"], tol_i, "dispersion")


@pytest.mark.parametrize("prec", [porta.F64, porta.F32])
def test_gradient_matches_oracle(strong, prec):
    freqs = np.arange(CFG.nfreq)
    atm, q, rays, seed, seed_sel = adj._problem(CFG, prec, freqs)
    ref = adj._oracle_grad(atm, q, rays, freqs, seed_sel, chunk=7)
    got = adj._gpu_grad(atm, q, prec, seed, stride=3)
    adj._compare(got, ref, prec, "dispersion")
