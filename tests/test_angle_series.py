"""The FP64 walk's sine and cosine of 2 pi (k/256 + t), |t| <= 1/512, restated on the
host: short series in t, rotated by the table's angle.  Tolerance 2^-52: the
table's entry, the series of the cosine and the result round once each (2^-54 for
numbers below 1, together 3/4 of it); the product with the sine of the small
angle, at most 0.0123, adds less than 1/50 of one of these.  (test_bm_tables.py
checks the logarithm and that k and t are exact.)
"""
import numpy as np


def _fma(a, b, c):
    # a long double's 64 bits hold the product of these series' factors to 2^-64: one rounding to double follows
    L = np.longdouble
    return (np.asarray(a, L) * np.asarray(b, L) + np.asarray(c, L)).astype(np.float64)


def test_sine_and_cosine_of_the_angle():
    h = float.fromhex
    rng = np.random.default_rng(5)
    t = np.concatenate([[0.0, 2.0 ** -9, -2.0 ** -9, 2.0 ** -53, -2.0 ** -53], rng.uniform(-2.0 ** -9, 2.0 ** -9, 4000)])
    z = t * t
    ps = _fma(h("-0x1.32d2cce62bd86p+6"), z, h("0x1.466bc6775aae2p+6"))
    ps = _fma(ps, z, h("-0x1.4abbce625be53p+5"))
    st = t * _fma(ps, z, h("0x1.921fb54442d18p+2"))
    pc = _fma(h("-0x1.55d3c7e3cbffap+6"), z, h("0x1.03c1f081b5ac4p+6"))
    pc = _fma(pc, z, h("-0x1.3bd3cc9be45dep+4"))
    ct = _fma(pc, z, 1.0)
    two_pi = 2 * np.longdouble(np.pi) + 2 * np.longdouble(h("0x1.1a62633145c07p-53"))
    for k in range(256):
        a = two_pi * k / 256
        sk, ck = np.sin(a).astype(np.float64), np.cos(a).astype(np.float64)
        s = _fma(sk, ct, ck * st)
        c = _fma(ck, ct, -(sk * st))
        angle = a + two_pi * t.astype(np.longdouble)
        assert np.max(np.abs(s - np.sin(angle))) < 2.0 ** -52
        assert np.max(np.abs(c - np.cos(angle))) < 2.0 ** -52
