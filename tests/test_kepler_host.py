"""The Kepler solver of the kernels (orbit.h, run on the CPU through
libcd4d_hostcheck.so) against bisection in extended precision: every solve ends
at the root, from the cold start and from the warm start of any step length.

Tolerance: E - M is exact, so f = E - e sin E - M carries the roundings of e sin E
(at most 1.5 ulp of 1 with the library sine's own), which the root's condition
1 / (1 - e cos E) magnifies, and E itself is rounded: 4 u (|E| + 1 / (1 - e cos E)),
u = 2^-52, leaves a factor of two."""
import ctypes
import os

import numpy as np
import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_1901_10475_amd", "libcd4d_hostcheck.so")
LD = np.longdouble


def _p(a):
    return a.ctypes.data_as(ctypes.c_void_p)


def _solve(M, dM, e):
    L = ctypes.CDLL(LIB)
    vp = ctypes.c_void_p
    L.hc_kepler.restype = None
    L.hc_kepler.argtypes = [ctypes.c_int64] + [vp] * 5
    M, dM, e = (np.ascontiguousarray(np.broadcast_to(v, M.shape), np.float64) for v in (M, dM, e))
    cold, warm = np.empty((len(M), 3)), np.empty((len(M), 3))
    L.hc_kepler(len(M), _p(M), _p(dM), _p(e), _p(cold), _p(warm))
    return cold, warm


def _roots(M, e):
    M, e = M.astype(LD), LD(e)
    lo, hi = M - e, M + e
    for _ in range(68):
        mid = (lo + hi) / 2
        up = mid - e * np.sin(mid) > M
        hi = np.where(up, mid, hi)
        lo = np.where(up, lo, mid)
    return (lo + hi) / 2


def _check(got, M, e, what):
    E = _roots(M, e)
    tol = 4 * 2.0 ** -52 * (np.abs(E) + 1 / (1 - LD(e) * np.cos(E)))
    for k, want in enumerate((E, np.sin(E), np.cos(E))):
        off = np.abs(got[:, k].astype(LD) - want) / tol
        w = int(np.argmax(off))
        assert off[w] <= 1, (what, "E sE cE".split()[k], float(off[w]), float(M[w]))


@pytest.mark.parametrize("e", [0.0, 0.1, 0.3, 0.5, 0.6, 0.65, 0.73, 0.85, 0.9, 0.95, 0.97, 0.99,
                               0.999])
def test_every_solve_ends_at_its_root(e):
    rng = np.random.default_rng(int(1000 * e))
    steps = [0.05, 0.1, 0.25, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0, 2 * np.pi, 12.0, 20.0]
    M = np.concatenate([rng.uniform(0, 2 * np.pi, 2500), rng.uniform(0, 40, 300),
                        np.arange(-3, 4) * np.pi,
                        np.outer([1, -1], 10.0 ** -np.arange(1, 9)).ravel()])
    for dM in steps:
        cold, warm = _solve(M, dM, e)
        _check(warm, M + dM, e, ("warm", dM))
    _check(cold, M, e, "cold")
