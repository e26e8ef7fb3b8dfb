"""Workspaces: a buffer of porta_workspace_size() bytes serves the call that it was asked for and
every call with fewer rays, a part of the ray range or a smaller batch.  CPU only: sizes, and
calls that end at the workspace check or, past it, for want of a device."""
import ctypes as C
import random

import numpy as np
import pytest

from paper_1307_4217_amd import inputs, porta, schedule


def _grid(nx, ny, nz, nmu, nchi, nfreq):
    cfg = inputs.Config("ws", nx, ny, nz, nmu, nchi, nfreq, True)
    q = inputs.make_quadrature(cfg)
    return porta.HostGrid(nx, ny, nz, 2000.0, 2000.0, np.linspace(0.0, 2000.0, nz), q.mu, q.wmu,
                          q.nchi, q.phi, q.wfreq)


# the last one: the range of 24 rays shares launches, which that of 28 does not
SIZES = [(37, 177, 82, 1, 8, 4), (16, 16, 32, 5, 8, 21), (64, 64, 49, 5, 8, 31),
         (200, 3, 2, 3, 7, 1), (150, 130, 64, 5, 16, 101)]


@pytest.mark.parametrize("kind", [porta.WS_SWEEP, porta.WS_ADJOINT, porta.WS_ADJOINT_CKPT])
@pytest.mark.parametrize("prec", [porta.F64, porta.F32])
@pytest.mark.parametrize("dims", SIZES)
def test_fewer_rays_need_no_more(dims, prec, kind):
    hg = _grid(*dims)
    nh = hg.nray_up
    rng = random.Random(str(dims))
    stride = min(5, hg.nz - 1)

    def size(**kw):
        return porta.workspace_size(hg, prec, kind, stride, porta.options(**kw))

    more = [{}] + ([{"stokes": 1}, {"faces": 1}, {"faces": 1, "faces_chunk": 1}]
                   if kind == porta.WS_SWEEP else [])
    for m in more:
        last = 0
        for n in range(1, nh + 1):   # batches
            now = size(ray_batch=n, **m)
            assert now >= last, (dims, m, n)
            last = now
        assert size(**m) == last
        for _ in range(60):   # ranges of a range
            a = rng.randrange(2 * nh)
            b = rng.randrange(a, 2 * nh)
            c = rng.randrange(a, b + 1)
            d = rng.randrange(c, b + 1)
            rb = rng.choice([0, rng.randint(1, nh)])
            whole = size(ray_first=a, ray_count=b + 1 - a, ray_batch=rb, **m)
            part = size(ray_first=c, ray_count=d + 1 - c, ray_batch=rb, **m)
            assert part <= whole, (dims, m, (a, b), (c, d), rb)


@pytest.mark.parametrize("dims,range_rays,ray_batch,prec", [
    ((150, 130, 64, 5, 16, 101), 28, 40, porta.F32),
    ((150, 130, 64, 5, 16, 101), 28, 40, porta.F64),
    ((37, 177, 82, 1, 8, 4), 3, 4, porta.F32)])
def test_interleaved_workspace_serves_every_range(dims, range_rays, ray_batch, prec):
    hg = _grid(*dims)
    s = schedule.InterleavedSweep(hg, prec, range_rays, ray_batch=ray_batch, device="meta")
    for o in s.range_opts + [s.down_opts]:
        assert porta.workspace_size(hg, prec, porta.WS_SWEEP, 1, o) <= s.workspace.numel()
    for o in s.range_opts:
        assert (porta.workspace_size(hg, prec, porta.WS_ADJOINT_CKPT, 1, o)
                <= s.workspace.numel())


def test_sharing_is_bounded():
    """The states of both hemispheres at once, where they share launches: at most 8 GiB more than
    those of a batch."""
    hg = _grid(256, 256, 3, 1, 8, 4000)
    state = 2 * 4000 * 65536 * 32
    for n in (1, 2, 3, 8):
        full = porta.workspace_size(hg, porta.F64, porta.WS_SWEEP, opts=porta.options(ray_batch=n))
        assert full <= n * state + (9 << 30), n


def test_planes_beyond_one_launch_go_plane_by_plane():
    """A launch holds fewer than 2^32 threads (J of planes of that size is reduced by launches of its
    own).  The partial sums of two planes more show where pairs are chosen."""
    def pairs(n, prec, nmu=1, nchi=1):
        hg = _grid(n, n, 3, nmu, nchi, 60)
        return (porta.workspace_size(hg, prec, porta.WS_SWEEP)
                > porta.workspace_size(hg, prec, porta.WS_SWEEP, opts=porta.options(block=256)))
    for prec in (porta.F32, porta.F64):
        assert not pairs(46000, prec)
        assert not pairs(16000, prec, 2, 8)
        assert pairs(8200, prec)
        assert pairs(16000, prec)


def _noalloc(hg, prec, opts=None):
    """Status of a no-alloc sweep on a machine without a GPU, which ends for want of a device once
    the size is accepted."""
    import torch
    if torch.cuda.device_count():
        pytest.skip("would run on the GPU")
    d = np.zeros(8).ctypes.data
    f = porta.Fields(d, d, d, 1.0, 1.0)
    return porta.lib().porta_fs_sweep_noalloc(
        C.byref(hg.grid), C.byref(hg.quad), C.byref(f), prec, porta.BILINEAR,
        C.byref(opts) if opts else None, d, 0, d, None)


@pytest.mark.parametrize("prec", [porta.F64, porta.F32])
@pytest.mark.parametrize("dims", [(1, 1, 7600, 5, 16, 1), (1, 1, 200000, 5, 16, 1),
                                  (3, 2, 30000, 5, 8, 2), (1, 1, 3000, 64, 32, 1)])
def test_noalloc_takes_long_columns(dims, prec):
    """The plane states and partial sums of these fit 64 MiB many times over; the rays' geometry
    on all layers would not."""
    assert _noalloc(_grid(*dims), prec) == porta.EDEVICE
    assert porta.workspace_size(_grid(*dims), prec, porta.WS_SWEEP) < 600 << 20


def test_noalloc_takes_what_its_acceptance_rule_takes():
    """First-face sweeps with many frequencies and few rays on wide planes, whose usual cut holds
    one frequency a block: the one of 321x64x2 with 68 frequencies needs 62 MiB by the rule and
    101 MiB in that cut.  Then any sweep: refused by the rule (its message gives the bytes) or
    not at all."""
    o = porta.options(ray_batch=1, faces=1)
    assert _noalloc(_grid(321, 64, 2, 1, 2, 68), porta.F32, o) == porta.EDEVICE
    rng = random.Random(7)
    taken = 0
    for _ in range(600):
        wide = rng.randint(64, 512)
        dims = (wide, rng.randint(1, 80), rng.choice([2, 2, 3, 9]), rng.randint(1, 3),
                rng.randint(1, 6), rng.randint(1, 100))
        if rng.random() < 0.3:
            dims = (dims[1], wide) + dims[2:]
        o = porta.options(ray_batch=rng.randint(0, 3), faces=rng.choice([1, 1, 0]))
        for prec in (porta.F64, porta.F32):
            status = _noalloc(_grid(*dims), prec, o)
            message = porta.lib().porta_last_error().decode()
            if status == porta.ENOMEM:
                assert "this sweep needs" in message, (dims, prec, o.ray_batch, message)
            else:
                assert status == porta.EDEVICE
                taken += 1
    assert taken > 200


def test_first_face_chunks_beyond_the_lds_stay_refused():
    """The option's limit: the rows of its frequencies in 64 KiB beside the tables of all
    frequencies (16 bytes each in FP64, 12 in FP32), and room for one frequency without it."""
    d = np.zeros(8).ctypes.data
    f = porta.Fields(d, d, d, 1.0, 1.0)

    def status(dims, prec, chunk):
        hg = _grid(*dims)
        return porta.lib().porta_fs_sweep(
            C.byref(hg.grid), C.byref(hg.quad), C.byref(f), prec, porta.BILINEAR,
            C.byref(porta.options(faces=1, faces_chunk=chunk)), d, 0, d, None, 0, 0, d, 16, None)

    wide = (321, 8, 2, 1, 2, 68)    # (64 KiB - 1088) / (408 rows of 32 bytes) = 4.9 in FP64
    assert status(wide, porta.F64, 4) == porta.ENOMEM
    assert status(wide, porta.F64, 5) == porta.EUNSUPPORTED
    many = (64, 8, 2, 1, 2, 4000)   # 1536 and 17536 bytes left; a row takes 2176
    for chunk, prec, want in ((0, porta.F64, porta.EUNSUPPORTED), (1, porta.F64, porta.EUNSUPPORTED),
                              (0, porta.F32, porta.ENOMEM), (8, porta.F32, porta.ENOMEM),
                              (9, porta.F32, porta.EUNSUPPORTED)):
        assert status(many, prec, chunk) == want, (chunk, prec)
