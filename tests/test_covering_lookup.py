"""The FP64 lookup of covering grids, restated on the host: with
q = fma(x, 1/d, -o/d - 1/2) and t its nearest integer, t is the voxel
floor((x - o) / d) wherever |q - t| stays within 1/2 less the rounding margin,
2^-51 times the sum of the magnitudes that enter (the bound of `covers` in
fk_api.cpp); the other points take the general lookup.  Points are placed a few
ulp from voxel faces, at spacings of every kind and grids up to 2^38 voxels from
the origin (the margin's limit of 2^-12 is reached on the way).  Without the
margin the test must find wrong voxels, so that it would see a bound too small.
"""
import ctypes

import numpy as np

_libm = ctypes.CDLL("libm.so.6")
_libm.fma.restype = ctypes.c_double
_libm.fma.argtypes = [ctypes.c_double] * 3
_fma = np.vectorize(_libm.fma, otypes=[np.float64])


def _grid(rng, far):
    """An axis: spacing, number of voxels, origin at about 2^far voxels from 0, and a box just inside."""
    d = float(np.exp(rng.uniform(np.log(1e-3), np.log(1e3))))
    if rng.random() < 0.25:
        d = 2.0 ** np.round(np.log2(d))
    n = int(rng.integers(1, 200))
    o = float(rng.choice([-1.0, 1.0]) * d * 2.0 ** (far + rng.random()))
    return d, n, o


def _points(rng, d, n, o, m):
    face = o + rng.integers(0, n + 1, m) * d
    x = np.concatenate([face + rng.integers(-6, 7, m) * np.spacing(np.abs(face)), o + n * d * rng.random(m // 4)])
    return x[(x >= o) & (x <= o + n * d)]


def _lookup(x, d, o):
    inv = 1.0 / d
    obh = float(-np.longdouble(o) / np.longdouble(d) - np.longdouble(0.5))
    q = _fma(x, inv, obh)
    t = np.rint(q)
    return t, np.abs(q - t)


def _margin(x, d, n, o):
    return 2.0 ** -51 * ((np.max(np.abs(x)) + abs(o)) / d + n + 2.0)


def test_nearest_integer_within_the_margin_is_the_voxel():
    rng = np.random.default_rng(7)
    wrong_without = used = 0
    reached = False
    for far in list(range(-6, 39, 2)) * 6:
        d, n, o = _grid(rng, far)
        x = _points(rng, d, n, o, 1500)
        t, dist = _lookup(x, d, o)
        voxel = np.floor((x - o) / d)
        margin = _margin(x, d, n, o)
        reached = reached or margin > 2.0 ** -12
        ok = dist <= 0.5 - margin
        assert np.array_equal(t[ok], voxel[ok]), (d, n, o)
        used += int(ok.sum())
        wrong_without += int(np.sum(t != voxel))
    assert reached and used > 10000 and wrong_without > 1000
