"""FP64 planes whose reduction of J is launches of its own, 64 nodes a block: a last block of one
node and of all but one, planes one by one and two by two, odd and even numbers of planes, ray
batches that leave one ray, intensity alone.  Against the sum of calls with one ray each, which
may be cut otherwise (1e-13, as between cuts elsewhere), and against the FP32 sweep of the same
inputs, which keeps the 16-node reduction (2e-5)."""
import numpy as np
import pytest

from gpu_common import Case, rounded
from paper_1307_4217_amd import inputs, porta

pytestmark = pytest.mark.gpu

# 128 x 240 is the smallest; 73 x 505 = 576 x 64 + 1 nodes, 3 x 12309 = 577 x 64 - 1; 60
# frequencies go two planes a launch
SIZES = [(128, 240, 3, 2, 8, 3), (73, 505, 3, 1, 5, 3), (3, 12309, 4, 1, 3, 2),
         (192, 192, 5, 1, 5, 60), (192, 192, 4, 1, 5, 60), (193, 200, 2, 2, 9, 2)]


@pytest.mark.parametrize("stokes", [4, 1])
@pytest.mark.parametrize("dims", SIZES)
def test_wide_reduction_equals_the_sum_over_rays(dims, stokes):
    import torch
    cfg = inputs.Config("wide", *dims, True)
    atm = rounded(inputs.make_atmosphere(cfg, seed=9), np.float32)
    q = inputs.make_quadrature(cfg)
    case = Case(atm, q, porta.F64)
    nh = case.hg.nray_up
    assert case.hg.nx * case.hg.ny >= 30720

    def sweep(case, prec, **kw):
        return porta.fs_sweep(case.hg, case.kappa, case.prop, case.emis, atm.i_bottom, atm.w2,
                              prec=prec, want_itop=False, opts=porta.options(stokes=stokes, **kw))[0]

    got = sweep(case, porta.F64)
    scale = float(got[0].abs().max())
    batches = sweep(case, porta.F64, ray_batch=nh - 1)
    one = sum(sweep(case, porta.F64, ray_first=r, ray_count=1) for r in range(2 * nh))
    for other in (batches, one):
        assert float((got - other).abs().max()) <= 1e-13 * scale
    single = sweep(Case(atm, q, porta.F32), porta.F32)
    assert float((got - single).abs().max()) <= 2e-5 * scale
    torch.cuda.synchronize()
