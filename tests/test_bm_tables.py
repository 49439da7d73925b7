"""The FP64 walk's table-driven logarithm and angle reduction, restated on the
host: the intervals of the logarithm's table and the angle's nearest 1/256 are
chosen from words by integer operations, so their edges are where they can go
wrong.

-2 ln u must stay within 2^-51 of the true value, relative: the interval's
2 ln v is a double (half an ulp, twice that where the series cancels half of
it), r = m v - 1, the series' last addition and the two of the exponent's term
round once each.  The angle's offset must be exact.
"""
import numpy as np

LOW, SHIFT = 0x3FE6B000, 13
BELOW1 = ((0x3FF00000 - LOW) >> SHIFT) - 1


def _double(hi, lo=0):
    return np.array([(int(hi) << 32) | int(lo)], dtype=np.uint64).view(np.float64)[0]


def _table():
    v = np.empty(128)
    g = np.empty(128)
    for j in range(128):
        c = _double(LOW + (j << SHIFT) + (1 << (SHIFT - 1)))
        v[j] = 1.0 / c
        g[j] = np.float64(2 * np.log(np.longdouble(v[j])))
    v[BELOW1], g[BELOW1] = float.fromhex("0x1.010108c28b78cp+0"), float.fromhex("0x1.00880f5e5822bp-7")
    return v, g


def _neg2_log(u):
    v, g = _table()
    bits = u.view(np.uint64)
    hw = (bits >> np.uint64(32)).astype(np.int64)
    t = (hw - LOW) & 0xFFFFFFFF
    k = t.astype(np.uint32).view(np.int32) >> 20
    m = (((hw - (t & 0xFFF00000)) & 0xFFFFFFFF).astype(np.uint64) << np.uint64(32) | (bits & np.uint64(0xFFFFFFFF))).view(np.float64)
    j = (t >> SHIFT) & 127
    L = np.longdouble
    r = (m.astype(L) * v[j].astype(L) - 1).astype(np.float64).astype(L)
    p = L(1) / 7
    for c in (L(-1) / 6, L(1) / 5, L(-1) / 4, L(1) / 3, L(-1) / 2):
        p = p * r + c
    l1p = (p * (r * r) + r).astype(np.float64)
    x = (-2 * l1p.astype(L) + g[j]).astype(np.float64)
    x = (k * -L(float.fromhex("0x1.a39ef35793c76p-32")) + x).astype(np.float64)
    return m, np.abs(r), (k * -L(float.fromhex("0x1.62e42fee00000p+0")) + x).astype(np.float64)


def test_logarithm_at_every_interval_edge_and_both_ends():
    rng = np.random.default_rng(1)
    edges = [_double(LOW + (j << SHIFT)) for j in range(129)]
    u = [2.0 ** -53, 2.0 ** -52, 1.0, np.nextafter(1.0, 0), 1.0 - 2.0 ** -30, 0.5, np.nextafter(0.5, 0)]
    for e in edges:
        for s in (1.0, 0.5, 0.25, 2.0 ** -40):
            x = e * s
            u += [x, np.nextafter(x, 0), np.nextafter(x, 2)]
    u = np.concatenate([u, rng.random(200000), 1.0 - rng.random(100000) / 200, np.exp(-36 * rng.random(100000))])
    u = u[(u > 0) & (u <= 1.0)]
    m, r, got = _neg2_log(u)
    assert np.all((m >= edges[0]) & (m < edges[-1]))
    assert np.max(r) < 0.0040
    want = -2 * np.log(u.astype(np.longdouble))
    assert np.all(got[u == 1.0] == 0.0)
    ok = want != 0
    assert np.max(np.abs((got[ok] - want[ok]) / want[ok])) < 2.0 ** -51


def test_uniform_and_angle_offset_are_exact():
    rng = np.random.default_rng(2)
    his = [0, 1, 0x7FFFFF, 0x800000, 0x800001, 0xFF7FFFFF, 0xFF800000, 0xFFFFFFFF] + [int(x) for x in rng.integers(0, 2 ** 32, 5000)]
    los = [0, 2047, 2048, 0xFFFFF800, 0xFFFFFFFF] + [int(x) for x in rng.integers(0, 2 ** 32, 40)]
    for hi in his:
        for lo in los[:5] + los[5 + hi % 40:7 + hi % 40]:
            n = ((hi << 21) | (lo >> 11)) + 1                                  # U = n 2^-53
            low = _double(0x3FE00000, (lo >> 11) + 1)
            assert (_double(0x41300000, hi) - (2.0 ** 20 + 0.5)) + low == n * 2.0 ** -53
            x = (hi + 0x800000) & 0xFFFFFFFF
            k, t = x >> 24, (_double(0x41300000, x & 0xFFFFFF) - (2.0 ** 20 + 0.5 + 2.0 ** -9)) + low
            whole = k if abs(n * 2.0 ** -53 - k / 256) <= 0.5 else k + 256      # modulo one turn
            assert int(t * 2.0 ** 53) == n - whole * 2 ** 45 and t * 2.0 ** 53 == int(t * 2.0 ** 53)
            assert abs(t) <= 2.0 ** -9
