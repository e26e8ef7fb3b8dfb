"""Plane steps cut into frequency chunks and shared by the two hemispheres: the launches of
small planes, against the oracle through the C ABI.

Sizes around the cut's edges: a chunk count that does not divide the frequencies, one
frequency, planes of less than a wavefront, of one wavefront plus a node and of several
blocks, an odd number of planes (both hemispheres' partial sums of J fall on the middle plane
in the same launch) and two planes.  Bars as for the whole sweep: FP64 1e-10 relative on I
and J, 1e-12 on Q/I, U/I, V/I; FP32 2e-5, 1e-7, 2e-5."""
import numpy as np
import pytest

from gpu_common import Case, compare_jkq, compare_stokes, rounded, up_rays
from paper_1307_4217_amd import inputs, porta

pytestmark = pytest.mark.gpu

SIZES = [(5, 3, 7, 2, 4, 1), (13, 5, 2, 1, 4, 22), (16, 16, 9, 3, 8, 23), (33, 20, 8, 2, 3, 5),
         (8, 8, 15, 2, 8, 101)]


def _case(dims, prec):
    cfg = inputs.Config("step", *dims, True)
    atm = inputs.make_atmosphere(cfg, seed=4)
    if prec == porta.F32:
        atm = rounded(atm, np.float32)
    return atm, inputs.make_quadrature(cfg)


@pytest.mark.parametrize("prec", [porta.F64, porta.F32])
@pytest.mark.parametrize("dims", SIZES)
def test_shared_chunked_steps_match_oracle(orc, dims, prec):
    atm, q = _case(dims, prec)
    ref = orc.fs_sweep(orc.OracleProblem(atm, q))
    case = Case(atm, q, prec)
    tol_i, tol_p = (1e-10, 1e-12) if prec == porta.F64 else (2e-5, 1e-7)
    nh = len(q.mu) * q.nchi
    for opts in (None, porta.options(ray_batch=max(1, nh - 1)), porta.options(block=64)):
        jkq, itop = case.sweep(opts=opts)
        compare_stokes(itop, up_rays(ref["itop"], q), tol_i, tol_p, str(dims))
        compare_jkq(jkq, ref["jkq"], tol_i, str(dims))
    # without J only the upward rays are swept, in other chunks: the same Stokes vectors
    _, alone = case.sweep(want_jkq=False)
    np.testing.assert_array_equal(alone, case.sweep()[1])


@pytest.mark.parametrize("prec", [porta.F64, porta.F32])
@pytest.mark.parametrize("dims", SIZES)
def test_shared_chunked_intensity_steps_match_oracle(orc, dims, prec):
    import dataclasses
    atm, q = _case(dims, prec)
    only = dataclasses.replace(atm, propmat=0 * atm.propmat, emis=np.concatenate(
        [atm.emis[:1], 0 * atm.emis[1:]]))
    ref = orc.fs_sweep(orc.OracleProblem(only, q))
    jkq, itop = Case(atm, q, prec).sweep(opts=porta.options(stokes=1))
    tol = 1e-10 if prec == porta.F64 else 2e-5
    want = up_rays(ref["itop"], q)[..., 0]
    assert np.abs(itop / want - 1).max() <= tol
    compare_jkq(jkq, ref["jkq"], tol, str(dims))


@pytest.mark.parametrize("dims", SIZES)
def test_ray_ranges_of_one_hemisphere_add_up(dims):
    """Ranges that hold rays of one hemisphere only, or unequal numbers of both: J of the
    calls adds up to the J of one call, the Stokes vectors are the same bit for bit."""
    atm, q = _case(dims, porta.F64)
    case = Case(atm, q, porta.F64)
    nh = len(q.mu) * q.nchi
    want_j, want_i = case.sweep()
    import torch
    jkq = torch.zeros((10, case.hg.N), dtype=torch.float64, device="cuda")
    itop = torch.zeros(want_i.shape, dtype=torch.float64, device="cuda")
    cuts = [0, nh - 1, nh + 2, 2 * nh - 1, 2 * nh]
    for a, b in zip(cuts, cuts[1:]):
        case.sweep(jkq=jkq, i_top=itop, accumulate=True,
                   opts=porta.options(ray_first=a, ray_count=b - a))
    np.testing.assert_array_equal(itop.cpu().numpy(), want_i)
    scale = np.abs(want_j[0]).max()
    assert np.abs(jkq.cpu().numpy() - want_j).max() <= 1e-13 * scale
