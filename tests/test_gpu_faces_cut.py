"""The cut of the first-face march into blocks of columns, sets of frequencies side by side
("ways") and frequencies in turn, against the oracle's first-face mode: one frequency; more
ways than frequencies and a last set that is smaller; rows of two and five wavefronts, which
leave room for four ways and for one; and more wavefronts than the chip holds, where a thread
takes several frequencies.  Bars as for the whole first-face sweep (test_gpu_faces)."""
import dataclasses

import numpy as np
import pytest

from gpu_common import Case, compare_jkq, compare_stokes, rounded, up_rays
from paper_1307_4217_amd import inputs, porta

pytestmark = pytest.mark.gpu

SIZES = [(5, 4, 5, 2, 4, 1), (6, 5, 4, 2, 4, 19), (100, 6, 4, 1, 4, 5), (300, 4, 3, 1, 4, 3),
         (4, 3, 3, 4, 16, 101)]


@pytest.mark.parametrize("prec", [porta.F64, porta.F32])
@pytest.mark.parametrize("dims", SIZES)
def test_first_face_cuts_match_oracle(orc, dims, prec):
    cfg = inputs.Config("cut", *dims, True)
    atm = inputs.make_atmosphere(cfg, seed=8)
    atm = dataclasses.replace(atm, lx=100.0 * cfg.nx, ly=100.0 * cfg.ny,
                              z=np.arange(cfg.nz) * 90.0)
    if prec == porta.F32:
        atm = rounded(atm, np.float32)
    q = inputs.make_quadrature(cfg)
    nh = len(q.mu) * q.nchi
    ref = orc.fs_sweep(orc.OracleProblem(atm, q, faces=1))
    case = Case(atm, q, prec)
    tol_i, tol_p = (1e-10, 1e-12) if prec == porta.F64 else (2e-5, 1e-7)
    for more in ({}, {"ray_batch": max(1, nh - 1)}, {"faces_chunk": 2}):
        jkq, itop = case.sweep(opts=porta.options(faces=1, **more))
        compare_stokes(itop, up_rays(ref["itop"], q), tol_i, tol_p, f"faces {dims} {more}")
        compare_jkq(jkq, ref["jkq"], tol_i, f"faces {dims} {more}")
