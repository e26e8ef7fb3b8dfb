"""Host build of the update's coefficients and source weights (no GPU), against extended
precision."""
import ctypes as C
import os

import numpy as np
import pytest

from paper_1307_4217_amd import build as pbuild


@pytest.fixture(scope="module")
def hm():
    if not os.path.exists(pbuild.HOSTTEST_LIB):
        pbuild.build_hostmath()
    L = C.CDLL(pbuild.HOSTTEST_LIB)
    L.hm_step_f32.argtypes = [C.c_float, C.POINTER(C.c_float)]
    L.hm_step_f64.argtypes = [C.c_double, C.POINTER(C.c_double)]
    return L


def _exact(tau):
    """e, psi'_M, psi'_O, omega_M, omega_O, omega_C, t E_1, t E_2, t E_3 in extended
    precision: the series of E_3 (terms below 1e-30) for tau < 2, else closed forms."""
    t = np.longdouble(tau)
    one = np.longdouble(1)
    if t < 2:
        term, e3, k = one / 6, np.longdouble(0), 0
        while abs(term) > 1e-30:
            e3 += term
            k += 1
            term = -term * t / (k + 3)
        e2 = one / 2 - t * e3
        e1 = one - t * e2
        e = one - t * e1
        return [e, t * (e1 - e2), t * e2, t * (e1 - 2 * e2 + 2 * e3), 2 * t * e3,
                t * (2 * e2 - 4 * e3), t * e1, t * e2, t * e3]
    e = np.exp(-t)
    return [e, (1 - e * (1 + t)) / t, (e + t - 1) / t, (2 - e * (t * t + 2 * t + 2)) / t**2,
            1 - 2 * (e + t - 1) / t**2, 2 * (t - 2 + e * (t + 2)) / t**2, 1 - e, (e + t - 1) / t,
            one / 2 - (e + t - 1) / t**2]


TAUS = np.concatenate([np.logspace(-9, 2, 400),
                       [0.999999, 1.0, 1.000001, 1.199999, 1.2, 1.200001, 0.1, 0.14, 0.18]])


def test_step_coefficients_f64(hm):
    """A few roundings of the recurrence (its differences lose at most a factor of 6 at small
    tau, 1/(1 - 1 + 1/3) and the like) or of the closed forms at tau >= 1 (omega_C loses a
    factor of 20 there): 40 ulp."""
    out = np.zeros(9)
    for tau in TAUS:
        hm.hm_step_f64(tau, out.ctypes.data_as(C.POINTER(C.c_double)))
        want = _exact(tau)
        for k in range(9):
            if want[k] < 1e-300:
                continue
            err = float(abs(np.longdouble(out[k]) / want[k] - 1))
            assert err < 40 * 2.0**-53, (tau, k, err)


def test_step_coefficients_f32(hm):
    """The same in single precision, at the rounded tau: 40 ulp."""
    out = np.zeros(9, np.float32)
    for tau in TAUS:
        t = np.float32(tau)
        hm.hm_step_f32(t, out.ctypes.data_as(C.POINTER(C.c_float)))
        want = _exact(t)
        for k in range(9):
            if want[k] < 1e-30:
                continue
            err = float(abs(np.longdouble(out[k]) / want[k] - 1))
            assert err < 40 * 2.0**-24, (tau, k, err)


def test_source_weights_give_the_sources(hm):
    """t E_1 A_1 + t E_2 A_2 + t E_3 A_3 with A_1 = S_M, A_2 = 2 (c_M - S_M), A_3 = 2 (S_M +
    S_O - 2 c_M) is omega_M S_M + omega_O S_O + omega_C c_M: to 16 ulp of the largest term."""
    rng = np.random.default_rng(5)
    out = np.zeros(9)
    for tau in TAUS:
        hm.hm_step_f64(tau, out.ctypes.data_as(C.POINTER(C.c_double)))
        w = [float(x) for x in _exact(tau)[3:6]]
        for _ in range(3):
            SM, SO, cM = rng.uniform(0.2, 2.0, 3)
            got = out[6] * SM + out[7] * 2 * (cM - SM) + out[8] * 2 * (SM + SO - 2 * cM)
            want = w[0] * SM + w[1] * SO + w[2] * cM
            big = out[6] * SM + abs(out[7] * 2 * (cM - SM)) + abs(out[8]) * 8
            assert abs(got - want) < 16 * 2.0**-53 * big, tau


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_lorentz_solve_matches_dense_solve(hm, prec):
    """(1 + p K') x = b and its transpose by the Lorentz-algebra route against a dense solve,
    K' entries up to 0.5.  K' then has norm < 1.5 and 1 + p K' condition < 10; each result is a
    sum of about 20 rounded terms of size <= 3 |b|: 400 ulp of the largest component."""
    rng = np.random.default_rng(9)
    ty, ct = (np.float64, C.c_double) if prec == "f64" else (np.float32, C.c_float)
    fn = getattr(hm, f"hm_lorentz_solve_{prec}")
    P = C.POINTER(ct)
    fn.argtypes = [P, P, ct, P, C.c_int, P]
    ulp = 2.0**-53 if prec == "f64" else 2.0**-24
    for trial in range(400):
        amp = (0.05, 0.5)[trial % 2]
        e, r = rng.uniform(-amp, amp, 3).astype(ty), rng.uniform(-amp, amp, 3).astype(ty)
        b, pp = rng.normal(size=4).astype(ty), ty(10.0 ** rng.uniform(-6, 0))
        K = np.array([[0, e[0], e[1], e[2]], [e[0], 0, r[2], -r[1]], [e[1], -r[2], 0, r[0]],
                      [e[2], r[1], -r[0], 0]], dtype=np.float64)
        A = np.eye(4) + float(pp) * K
        for sgn, M in ((1, A), (-1, A.T)):
            want = np.linalg.solve(M, b.astype(np.float64))
            x = np.zeros(4, ty)
            fn(e.ctypes.data_as(P), r.ctypes.data_as(P), pp, b.ctypes.data_as(P), sgn,
               x.ctypes.data_as(P))
            assert np.abs(x - want).max() <= 400 * ulp * np.abs(want).max()


def _solve_longdouble(M, b):
    """Gaussian elimination with row pivoting in extended precision."""
    A = np.concatenate([M, b[:, None]], axis=1).astype(np.longdouble)
    n = len(b)
    for c in range(n):
        k = c + int(np.argmax(np.abs(A[c:, c])))
        A[[c, k]] = A[[k, c]]
        for r in range(c + 1, n):
            A[r] -= A[c] * (A[r, c] / A[c, c])
    x = np.zeros(n, np.longdouble)
    for r in range(n - 1, -1, -1):
        x[r] = (A[r, n] - A[r, r + 1:n] @ x[r + 1:]) / A[r, r]
    return x


@pytest.mark.parametrize("disp", [0.5, 3.0, 10.0, 30.0, 100.0, 1000.0])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_lorentz_solve_under_strong_dispersion(hm, prec, disp):
    """The same solve where the dispersion exceeds the absorption by up to 1000, with dichroism
    up to 0.3.  No part of the solution exceeds about |b| there (the inverse damps what is
    perpendicular to the dispersion), and each is a sum of at most 20 terms of that size with
    some ten roundings each, so the error stays below 100 ulp of |b| at any dispersion; a form
    that takes 1 + p^2 r.r apart again loses p^2 r.r ulp."""
    rng = np.random.default_rng(17)
    ty, ct = (np.float64, C.c_double) if prec == "f64" else (np.float32, C.c_float)
    fn = getattr(hm, f"hm_lorentz_solve_{prec}")
    P = C.POINTER(ct)
    fn.argtypes = [P, P, ct, P, C.c_int, P]
    ulp = 2.0**-53 if prec == "f64" else 2.0**-24
    for trial in range(300):
        e, r = rng.uniform(-0.3, 0.3, 3).astype(ty), rng.normal(size=3)
        r = (disp * r / np.linalg.norm(r)).astype(ty)
        b, pp = rng.normal(size=4).astype(ty), ty((0.9, 0.5, 0.1)[trial % 3])
        eL, rL = e.astype(np.longdouble), r.astype(np.longdouble)
        K = np.array([[0, eL[0], eL[1], eL[2]], [eL[0], 0, rL[2], -rL[1]],
                      [eL[1], -rL[2], 0, rL[0]], [eL[2], rL[1], -rL[0], 0]], dtype=np.longdouble)
        A = np.eye(4, dtype=np.longdouble) + np.longdouble(pp) * K
        for sgn, M in ((1, A), (-1, A.T)):
            want = _solve_longdouble(M, b.astype(np.longdouble))
            x = np.zeros(4, ty)
            fn(e.ctypes.data_as(P), r.ctypes.data_as(P), pp, b.ctypes.data_as(P), sgn,
               x.ctypes.data_as(P))
            assert np.abs(x - want).max() <= 100 * ulp * np.abs(b).max(), (disp, trial, sgn)


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_sources_of_steep_and_thick_steps(hm, prec):
    """omega_M S_M + omega_O S_O + omega_C c_M as the kernels form it, where S_M and S_O differ
    by up to 10^8 and the step is up to 10^6 thick: three positive terms, each of a coefficient
    within 40 ulp and one more rounding, added with two: 44 ulp of their sum."""
    fn = getattr(hm, f"hm_sources_{prec}")
    ty, ct = (np.float64, C.c_double) if prec == "f64" else (np.float32, C.c_float)
    fn.argtypes, fn.restype = [ct] * 4, ct
    ulp = 2.0**-53 if prec == "f64" else 2.0**-24
    for tau in np.concatenate([TAUS[TAUS > 1e-6], [1e3, 1e4, 1e5, 1e6]]).astype(ty):
        w = _exact(tau)[3:6]
        for steep in (1.0, 1e2, 1e4, 1e6, 1e8):
            for SM, SO in ((steep, 0.7), (0.7, steep)):
                for part in (0.0, 0.3, 1.0):   # the control point between the two
                    S = np.array([SM, SO, SM + part * (SO - SM)]).astype(ty)
                    want = sum(c * np.longdouble(v) for c, v in zip(w, S))
                    assert abs(np.longdouble(fn(tau, *S)) - want) <= 44 * ulp * want, (tau, S)


@pytest.mark.parametrize("half", [0.0, 0.5])
def test_cell_shift_stays_on_the_axis(hm, half):
    """Node offsets in [0, n], which the kernels add to an index and wrap once, for every
    displacement: within reach, at and around whole periods, beyond 2^53 cells, where the period
    cannot be taken off exactly, and not finite."""
    hm.hm_cell_shift.argtypes = [C.c_double, C.c_int, C.c_double, C.POINTER(C.c_double)]
    t = C.c_double()
    rng = np.random.default_rng(21)
    for n in (1, 2, 3, 7, 64, 250, 4093):
        near = [k * n * (1 + d * 2.0**-52) for k in (-9, -1, 0, 1, 2, 17, 1023) for d in (-1, 0, 1)]
        far = [s * 10.0**e for s in (-1, 1, -1.7, 1.3) for e in range(14, 308, 7)]
        inside = (list(rng.uniform(-20 * n, 20 * n, 300)) +
                  [k + d for k in range(-2, 3) for d in (-0.5, 0.0, 0.5)])
        for u in near + far + inside + [np.inf, -np.inf, np.nan]:
            f = hm.hm_cell_shift(u, n, half, C.byref(t))
            assert 0 <= f <= n, (u, n, f)
            if abs(u) < 1e6:
                # the place itself, up to the rounding of the reduced displacement
                off = (f + t.value - u) / n
                assert abs(off - round(off)) * n <= 4e-16 * (abs(u) + n), (u, n, f, t.value)
                assert -half <= t.value <= 1 - half
