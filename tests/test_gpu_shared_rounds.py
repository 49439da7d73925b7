"""GPU: launches that give every wavefront a few walks run them in shared
drain rounds; the number of live walks decides how a round is divided (3 lanes
per walk up to 16 walks, 21 with the bridge test, the walks' own lanes beyond, and as many macro-steps as
the block slots hold).  At the edges of those ranges every walk's
record must equal the oracle's in FP64 (1e-12 of the mean |u|, step counts
exactly), and in every precision, bit for bit, what a full launch records.
"""
import functools

import numpy as np
import pytest

import oracle
from paper_1709_07469_amd import workloads as W
from gpu_helpers import compare_walks, gpu_solve, say

pytestmark = pytest.mark.gpu

WAVES = 256          # one 64-thread block per compute unit
CAPS = (1, 2, 3, 16, 17, 21, 22, 32, 33, 42, 43, 63)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _problem(name, n, precision):
    if name == "box":          # a grid, a prism and a ball at once, data read on the faces
        pr = W.cfg3(n, precision=precision, n=32)
        return pr.replace(stations=pr.stations[100:101], dt=4e-3, exit_rule=W.EXIT_INTERSECT, max_steps=150,
                          prisms=np.array([[-0.9, -0.9, 0.0, 0.3, 0.4, 0.6, 50.0]]),
                          spheres=np.array([[0.1, 0.2, 0.3, 0.4, 70.0]]))
    ball = W.paper_ball(stations=np.array([[0.05, 0.05, 0.2]]), dt_paper=0.1, paths_per_station=n,
                        precision=precision)
    return ball.replace(exit_rule=W.EXIT_BRIDGE, prisms=np.array([[-3.0, -2.0, -4.0, 3.0, 4.0, 5.0, 2e12]]))


@functools.lru_cache(maxsize=None)
def _full(name, precision):
    """The walks of a launch that fills its wavefronts: 64 per wavefront and more."""
    from paper_1709_07469_amd import fkgrav as F
    keep = F.fk_get_launch(precision)
    try:
        F.fk_set_launch(precision, 64, 1, 32)
        _, v, s = gpu_solve(_problem(name, WAVES * 80, precision), 0)
    finally:
        F.fk_set_launch_dict(precision, keep)
    return v[0], s[0]


@functools.lru_cache(maxsize=None)
def _oracle(name):
    _, u, steps = oracle.solve(_problem(name, WAVES * max(CAPS), W.PREC_F64), 0)
    return u[0], steps[0]


@pytest.mark.parametrize("precision", [W.PREC_F64, W.PREC_MIXED_F64ACC, W.PREC_MIXED_KAHAN])
@pytest.mark.parametrize("name", ["box", "ball"])
def test_few_walks_per_wavefront_record_the_same_walks(name, precision):
    from paper_1709_07469_amd import fkgrav as F
    fv, fs = _full(name, precision)
    keep = F.fk_get_launch(precision)
    try:
        F.fk_set_launch(precision, 64, 1, 32)
        for cap in CAPS:
            n = WAVES * cap - (3 if cap > 1 else 0)
            say("walks per wavefront", cap, "precision", precision, name)
            _, v, s = gpu_solve(_problem(name, n, precision), 0)
            assert v[0].tobytes() == fv[:n].tobytes() and s[0].tobytes() == fs[:n].tobytes(), (cap, precision)
            if precision == W.PREC_F64:
                u, steps = _oracle(name)
                live = u[:n][np.isfinite(u[:n])]
                r = compare_walks(v[0], s[0], u[:n], steps[:n], np.mean(np.abs(live)))
                assert r["step_mismatch"] == 0 and r["value_mismatch"] == 0 and r["capped_nan"], (cap, r)
    finally:
        F.fk_set_launch_dict(precision, keep)
