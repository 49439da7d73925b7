"""The logarithm of the prism closed form.  ln_ratio replaces a quotient whose
logarithm is not wanted (a term with a zero prefactor) by 1, and passes every
other one to the table logarithm, which takes the exponent from the number's
high word and so needs a positive normal number.  Every quotient that the
source's guard lets through must therefore have its logarithm, from the smallest
on (a subnormal number's would be off by up to 36); the largest is the largest
finite number.  The logarithm is the one of test_bm_tables.py: relative error
below 2^-51.
"""
import os
import re

import numpy as np

from test_bm_tables import _neg2_log

SOURCE = os.path.join(os.path.dirname(__file__), "..", "paper_1709_07469_amd", "csrc", "fk_device.hpp")


def _number(text):
    return float.fromhex(text) if "p" in text else float(text)


def _accepted():
    """The least and the greatest quotient that ln_ratio's guard passes on."""
    with open(SOURCE) as f:
        m = re.search(r"x = \(x (>=?) (\S+) && x <= (\S+)\) \? x : 1\.0;", f.read())
    least = _number(m.group(2))
    return (np.nextafter(least, 1.0) if m.group(1) == ">" else least), _number(m.group(3))


def test_logarithm_of_every_accepted_quotient():
    least, greatest = _accepted()
    rng = np.random.default_rng(4)
    u = np.concatenate([[least, np.nextafter(least, 1.0), 3 * least, 2.0 ** -1022, 1.0, 2.0, greatest,
                         np.nextafter(greatest, 0.0)], np.exp(rng.uniform(np.log(2.0 ** -1021), np.log(greatest), 20000))])
    _, _, got = _neg2_log(u)
    want = -2 * np.log(u.astype(np.longdouble))
    ok = want != 0
    assert np.all(got[~ok] == 0.0)
    assert np.max(np.abs((got[ok] - want[ok]) / want[ok])) < 2.0 ** -51
