"""A plane of more than 2^27 nodes, whose reduction of J no longer fits a plane step's launch
(16 nodes a block of 256 threads, for both hemispheres) and goes in launches of its own: columns
that are all alike, against the same columns on a plane of 16x16."""
import numpy as np
import pytest

from gpu_common import require_gpu
from paper_1307_4217_amd import inputs, porta

pytestmark = pytest.mark.gpu


def test_intensity_on_a_plane_of_more_than_2_27_nodes():
    torch = require_gpu()
    n, nz = 11600, 2
    assert n * n > 1 << 27
    cfg = inputs.Config("large", 16, 16, nz, 1, 1, 1, False)
    q = inputs.make_quadrature(cfg)
    kap, eps = np.array([0.8, 0.3]), np.array([1.1, 0.7])
    got = []
    for size in (16, n):
        hg = porta.HostGrid(size, size, nz, 2.0 * size, 2.0 * size, np.array([0.0, 1.5]), q.mu,
                            q.wmu, q.nchi, q.phi, q.wfreq)
        f = [torch.tensor(v, dtype=torch.float32, device="cuda").repeat_interleave(size * size)
             for v in (kap, kap * eps)]
        j, it = porta.fs_sweep(hg, f[0], f[0], f[1], 0.9, 0.0, prec=porta.F32,
                               opts=porta.options(stokes=1))
        torch.cuda.synchronize()
        got.append((j.view(10, nz, size * size), it.view(-1)))
    (j0, i0), (j1, i1) = got
    assert float((i1 / i0[0] - 1).abs().max()) <= 2e-5
    for c in range(10):
        for k in range(nz):
            want = float(j0[c, k, 0])
            tol = 2e-5 * abs(float(j0[0, k, 0]))
            lo, hi = float(j1[c, k].min()), float(j1[c, k].max())
            assert want - tol <= lo and hi <= want + tol, (c, k, want, lo, hi)
