"""Launches of two planes (large sweeps) against one plane per launch (a `block` in the
options), which the other tests hold against the oracle.

A node's Stokes vectors come from the same operations on either path: FP32 Stokes vectors and
J are the same bit for bit, in FP64 to the roundings of J's sums and of set-up shared
differently (1e-13).  Sizes: planes of exactly one 16x14 tile, ragged tiles, planes narrower
than a tile in one direction, nz of 2 to 6 (the last launch holds one plane or two), one
frequency, and ray batches that leave a smaller last one.  Which sizes go in pairs depends on
the number of frequencies too; CHOSEN and SHARED are sizes that do, the latter with both
hemispheres in a launch (planes 2 to 5: the hemispheres' sums meet on a plane of J in the
middle of the march, at its end, in different positions of a launch)."""
import numpy as np
import pytest

from gpu_common import Case, compare_jkq, compare_stokes, rounded, up_rays
from paper_1307_4217_amd import inputs, porta

pytestmark = pytest.mark.gpu

# (nx, ny, nz, inclinations, azimuths, frequencies): tiles of 256 nodes times rays > 2048
SIZES = [(16, 14, 5, 16, 129, 2), (33, 29, 4, 8, 90, 3), (100, 3, 2, 8, 130, 1),
         (2, 161, 6, 8, 130, 2)]


def _case(dims, prec):
    cfg = inputs.Config("pair", *dims, True)
    atm = inputs.make_atmosphere(cfg, seed=2)
    if prec == porta.F32:
        atm = rounded(atm, np.float32)
    q = inputs.make_quadrature(cfg)
    return atm, q, Case(atm, q, prec)


def _same(got, want, prec, what):
    if prec == porta.F32:
        np.testing.assert_array_equal(got, want, err_msg=what)
    else:
        assert np.abs(got - want).max() <= 1e-13 * np.abs(want).max(), what


@pytest.mark.parametrize("prec", [porta.F64, porta.F32])
@pytest.mark.parametrize("dims", SIZES)
def test_two_planes_a_launch_equal_one(dims, prec):
    atm, q, case = _case(dims, prec)
    nh = len(q.mu) * q.nchi
    for more in ({}, {"ray_batch": nh - 3}, {"ray_first": 2, "ray_count": 2 * nh - 5},
                 {"control": 1}):
        want = case.sweep(opts=porta.options(block=256, **more))
        got = case.sweep(opts=porta.options(**more))
        for a, b, n in zip(got, want, ("J", "I_top")):
            _same(a, b, prec, f"{dims} {more} {n}")
    _same(case.sweep(want_jkq=False)[1], case.sweep(opts=porta.options(block=256))[1], prec,
          f"{dims} without J")


@pytest.mark.parametrize("prec", [porta.F64, porta.F32])
def test_two_planes_a_launch_match_oracle(orc, prec):
    dims = (33, 29, 4, 4, 180, 1)
    atm, q, case = _case(dims, prec)
    ref = orc.fs_sweep(orc.OracleProblem(atm, q))
    jkq, itop = case.sweep()
    tol_i, tol_p = (1e-10, 1e-12) if prec == porta.F64 else (2e-5, 1e-7)
    compare_stokes(itop, up_rays(ref["itop"], q), tol_i, tol_p, str(dims))
    compare_jkq(jkq, ref["jkq"], tol_i, str(dims))


@pytest.mark.parametrize("stride", [1, 2, 3])
def test_two_planes_a_launch_keep_checkpoints(stride):
    """The planes kept for the adjoint, which may be the first or the second of a launch."""
    import torch
    from paper_1307_4217_amd.porta import checkpoint_size, fs_sweep
    atm, q, case = _case((33, 29, 6, 8, 90, 2), porta.F32)
    kept = []
    for opts in (porta.options(block=256), porta.options()):
        ck = torch.zeros(checkpoint_size(case.hg, porta.F32, stride, opts), dtype=torch.uint8,
                         device="cuda")
        fs_sweep(case.hg, case.kappa, case.prop, case.emis, atm.i_bottom, atm.w2, prec=porta.F32,
                 opts=opts, checkpoints=ck, checkpoint_stride=stride)
        torch.cuda.synchronize()
        kept.append(ck.cpu().numpy())
    np.testing.assert_array_equal(kept[1], kept[0])


CHOSEN = [(16, 14, 3, 16, 129, 60), (47, 41, 4, 8, 45, 60), (30, 13, 2, 8, 130, 60),
          (15, 42, 5, 8, 90, 60)]
SHARED = [(32, 28, 5, 5, 8, 31), (32, 28, 4, 5, 8, 31), (48, 40, 2, 3, 4, 40),
          (48, 42, 3, 3, 4, 40), (30, 13, 7, 8, 10, 41)]


@pytest.mark.parametrize("dims,prec", [(d, p) for d in CHOSEN for p in (porta.F64, porta.F32)] +
                         [(d, porta.F64) for d in SHARED])
def test_chosen_pairs_equal_one_plane_a_launch(dims, prec):
    import torch
    atm, q, case = _case(dims, prec)
    nh = len(q.mu) * q.nchi
    for more in ({}, {"ray_batch": nh - 1}, {"ray_first": 2, "ray_count": 2 * nh - 5},
                 {"ray_first": nh, "ray_count": nh}):
        out, size = [], []
        for opts in (porta.options(block=256, **more), porta.options(**more)):
            size.append(porta.workspace_size(case.hg, prec, porta.WS_SWEEP, opts=opts))
            itop = torch.zeros((nh, case.hg.nfreq, atm.ny, atm.nx, 4), dtype=case.dt,
                               device="cuda")   # rays out of the range are not written
            out.append(porta.fs_sweep(case.hg, case.kappa, case.prop, case.emis, atm.i_bottom,
                                      atm.w2, prec=prec, opts=opts, i_top=itop))
        torch.cuda.synchronize()
        if not more:
            assert size[0] != size[1]   # partial sums of two planes: the pairs are chosen
        for want, got, n in zip(*out, ("J", "I_top")):
            if prec == porta.F32:
                assert torch.equal(got, want), (dims, more, n)
            else:
                scale = float(want.abs().max())
                assert float((got - want).abs().max()) <= 1e-13 * scale, (dims, more, n)


def test_shared_pairs_match_oracle(orc):
    dims = (32, 28, 5, 5, 8, 31)
    atm, q, case = _case(dims, porta.F64)
    ref = orc.fs_sweep(orc.OracleProblem(atm, q))
    jkq, itop = case.sweep()
    compare_stokes(itop, up_rays(ref["itop"], q), 1e-10, 1e-12, str(dims))
    compare_jkq(jkq, ref["jkq"], 1e-10, str(dims))


def test_many_frequencies_go_plane_by_plane():
    """2500 frequencies, whose FP64 tables leave no room in LDS for the tiles of a pair."""
    atm, q, case = _case((16, 14, 3, 4, 10, 2500), porta.F64)
    opts = porta.options(block=256)
    assert (porta.workspace_size(case.hg, porta.F64, porta.WS_SWEEP) ==
            porta.workspace_size(case.hg, porta.F64, porta.WS_SWEEP, opts=opts))
    for a, b in zip(case.sweep(), case.sweep(opts=opts)):
        np.testing.assert_array_equal(a, b)
