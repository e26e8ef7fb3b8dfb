"""FP32 planes whose reduction of J is launches of its own, a node a thread: the sums of the rays
in the order of the enumeration, bitwise those of the blocks of small planes.  A periodic plane is
laid out several times side by side, so that every copy has the small plane's Stokes vectors,
but for places where the period rounds a ray's offset to another last bit: J of the top plane
bitwise where the emergent Stokes vectors of every ray are, J of the other planes to 1e-6 (a few
roundings of 6e-8).  Around the lines of the rule for up to 3, up to 6 and more rays: a ragged last
block, an odd and an even number of planes, two planes a launch, batches whose last has fewer
rays, a range of rays, and intensity alone."""
import numpy as np
import pytest

from gpu_common import require_gpu
from paper_1307_4217_amd import inputs, porta

pytestmark = pytest.mark.gpu

# plane, copies in x and y, nz, inclinations, azimuths, frequencies, options
CASES = [((64, 64), (4, 4), 5, 1, 1, 3, {}), ((64, 64), (4, 4), 4, 1, 3, 2, {}),
         ((33, 31), (9, 8), 4, 1, 2, 2, {}), ((33, 31), (9, 9), 3, 1, 3, 2, {}),
         ((64, 80), (4, 4), 3, 1, 6, 2, {}), ((64, 64), (8, 4), 5, 1, 7, 2, {}),
         ((43, 64), (8, 6), 4, 3, 12, 2, {}), ((64, 64), (8, 4), 4, 2, 8, 40, {}),
         ((64, 64), (4, 4), 4, 1, 5, 2, {"ray_batch": 3}),
         ((64, 64), (4, 4), 3, 1, 5, 3, {"ray_first": 3, "ray_count": 4})]


@pytest.mark.parametrize("stokes", [4, 1])
@pytest.mark.parametrize("plane,copies,nz,nmu,nchi,nfreq,options", CASES)
def test_wide_fp32_reduction_is_bitwise_that_of_small_planes(plane, copies, nz, nmu, nchi, nfreq,
                                                             options, stokes):
    torch = require_gpu()
    nx, ny = plane
    cfg = inputs.Config("wide", nx, ny, nz, nmu, nchi, nfreq, True)
    atm, q = inputs.make_atmosphere(cfg, seed=6), inputs.make_quadrature(cfg)
    out = []
    for cx, cy in ((1, 1), copies):
        hg = porta.HostGrid(nx * cx, ny * cy, nz, float(nx * cx), float(ny * cy), atm.z, q.mu,
                            q.wmu, q.nchi, q.phi, q.wfreq)
        f = [torch.tensor(np.asarray(v, np.float32).reshape(-1, nz, ny, nx), device="cuda")
             .tile(1, 1, cy, cx).reshape(-1).contiguous()
             for v in (atm.kappa, atm.propmat, atm.emis)]
        j, it = porta.fs_sweep(hg, *f, atm.i_bottom, atm.w2, prec=porta.F32,
                               opts=porta.options(stokes=stokes, **options))
        out.append((j.view(10, nz, ny * cy, nx * cx),
                    it.view(-1, nfreq, ny * cy, nx * cx, stokes)[options.get("ray_first", 0):]))
    (j0, i0), (j1, i1) = out
    j0, i0 = j0.tile(1, 1, copies[1], copies[0]), i0.repeat(1, 1, copies[1], copies[0], 1)
    scale = float(j0[0].abs().max())
    assert scale > 0 and float((j0 - j1).abs().max()) <= 1e-6 * scale
    same = (i0 == i1).all(dim=4).all(dim=1).all(dim=0)
    assert float(same.float().mean()) > 0.99
    assert torch.equal(j0[:, -1][:, same], j1[:, -1][:, same])
