"""Rays displaced by 10^17 cells and more between two planes (a period of 10^-14 on planes 1000
apart), whose place on the period has no meaning left but is read all the same: on planes that
are alike everywhere the outputs do not depend on it, and equal those of an ordinary period."""
import numpy as np
import pytest

from gpu_common import require_gpu
from paper_1307_4217_amd import inputs, porta

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [porta.F64, porta.F32])
def test_displacements_beyond_the_integers(prec):
    torch = require_gpu()
    nx, ny, nz = 7, 6, 5
    q = inputs.make_quadrature(inputs.Config("shift", nx, ny, nz, 3, 4, 4, False))
    rng = np.random.default_rng(4)
    dt = torch.float64 if prec == porta.F64 else torch.float32

    def field(rows, lo, hi):
        v = torch.as_tensor(rng.uniform(lo, hi, (rows, nz)), dtype=dt, device="cuda")
        return v.repeat_interleave(nx * ny, dim=1).contiguous()

    kappa, prop, emis = field(1, 1e-3, 4e-3), field(6, -1e-4, 1e-4), field(6, -1e-4, 1e-4)
    emis[0] = field(1, 1e-3, 3e-3)[0]
    got = []
    for period in (2000.0, 1e-14):
        hg = porta.HostGrid(nx, ny, nz, period, period, np.linspace(0.0, 4000.0, nz), q.mu, q.wmu,
                            q.nchi, q.phi, q.wfreq)
        out = []
        for interp, opts in ((porta.BILINEAR, None), (porta.BILINEAR, porta.options(stokes=1)),
                             (porta.BEZIER2D, None)):
            j, it = porta.fs_sweep(hg, kappa, prop, emis, 1.0, 1.0, prec=prec, interp=interp,
                                   opts=opts)
            out += [j, it]
            if opts is None:
                g = porta.fs_adjoint(hg, kappa, prop, emis, 1.0, it, 1.0, prec=prec, interp=interp,
                                     checkpoint_stride=2)
                # a shift moves a gradient from node to node of a plane, not its sum
                out += [x.view(-1, nz, nx * ny).double().sum(dim=2) for x in g]
        torch.cuda.synchronize()
        got.append(out)
    assert len(got[0]) == 12
    for k, (a, b) in enumerate(zip(*got)):
        # (J and I_top of three calls, three gradients after the first and the last)
        grad = k in (2, 3, 4, 9, 10, 11)
        tol = 1e-10 if prec == porta.F64 else (1e-4 if grad else 2e-5)
        assert torch.isfinite(b).all(), k
        assert float((a - b).abs().max()) <= tol * float(a.abs().max()), k
