"""GPU: grids that cover their box take a lookup without clamps and tests for the
macro-steps that stay inside (the covering loop).  A batch takes that loop only
when every problem's grid covers its box, so each form of grid is walked twice:
in a batch of its own kind, and in a batch with a problem whose grid does not
cover (the general loop).  Every walk's record must be the same, bit for bit,
over spacings, ragged and single-voxel axes, grids larger than the box or short
of it by less than the rule allows, boxes far from the origin, grids by levels,
bodies beside the grid, both exit rules and walks cut at max_steps.
"""
import numpy as np
import pytest

from paper_1709_07469_amd import workloads as W
from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _grid(n, origin, spacing, lo=(-1, -1, -1), hi=(1, 1, 1), **kw):
    """Random densities of 40 values on a grid over the box [lo, hi]; two stations, one 1e-3 from a face."""
    rng = np.random.Generator(np.random.PCG64(11))
    rho = rng.choice(rng.uniform(-5, 5, 40).astype(np.float32), size=tuple(n[::-1]))
    lo, hi = np.asarray(lo, float), np.asarray(hi, float)
    w = hi - lo
    st = np.stack([lo + 0.45 * w, np.array([hi[0] - 1e-3 * w[0], lo[1] + 0.3 * w[1], lo[2] + 0.6 * w[2]])])
    return W.Problem(box_lo=lo, box_hi=hi, stations=st, dt=4e-3 * float(np.min(w)) ** 2 / 4, paths_per_station=9001,
                     seed=3, G=1.0, rho=rho, grid_origin=np.asarray(origin, float),
                     grid_spacing=np.asarray(spacing, float), bc_kind=W.BC_QUADRATIC,
                     bc_data=np.array([1.0, 0.1, 0.2, 0.3, 0.5, 0.0, 0.0, 0.4, 0.0, 0.3]), **kw)


FORMS = {
    "powers of two": lambda: _grid((32, 64, 16), (-1, -1, -1), (2 / 32, 2 / 64, 2 / 16)),
    "general spacings": lambda: _grid((33, 29, 27), (-1, -1, -1), (2 / 33, 2 / 29, 2 / 27)),
    "beyond the box": lambda: _grid((41, 37, 50), (-1.3, -1.07, -2.0), (2.7 / 41, 2.3 / 37, 4 / 50)),
    "short of the box": lambda: _grid((50, 50, 50), (-1, -1 + 1 / 300, -1), (2 / 50, (2 - 1 / 300) / 50, 1.994 / 50)),
    "far from the origin": lambda: _grid((30, 31, 32), (1000, -2000, 500), (2 / 30, 3 / 31, 2 / 32), (1000, -2000, 500),
                                         (1002, -1997, 502)),
    "single voxels": lambda: _grid((1, 40, 1), (-1, -1, -1), (2, 2 / 40, 2)),
    "bodies beside": lambda: _grid((24, 23, 22), (-1, -1, -1), (2 / 24, 2 / 23, 2 / 22),
                                   prisms=np.array([[-0.5, -0.5, -0.5, 0.2, 0.9, 0.3, 7.0]]),
                                   spheres=np.array([[0.2, 0.1, 0.3, 0.4, -3.0]])),
    "cut at max_steps": lambda: _grid((33, 29, 27), (-1, -1, -1), (2 / 33, 2 / 29, 2 / 27), max_steps=37),
    "data on the faces": lambda: _grid((33, 29, 27), (-1, -1, -1), (2 / 33, 2 / 29, 2 / 27),
                                       exit_rule=W.EXIT_INTERSECT),
}


@pytest.mark.parametrize("precision", [W.PREC_F64, W.PREC_MIXED_F64ACC, W.PREC_MIXED_KAHAN])
@pytest.mark.parametrize("levels", [False, True])
def test_covering_loop_equals_general_loop(precision, levels):
    from paper_1709_07469_amd import fkgrav as F
    probs = [f().replace(precision=precision, grid_levels=levels, problem_id=m) for m, f in enumerate(FORMS.values())]
    # half a grid: most of the box lies outside it
    other = _grid((16, 16, 16), (-1, -1, -1), (1 / 16,) * 3).replace(precision=precision, grid_levels=levels,
                                                                     problem_id=99, paths_per_station=64)
    keep = F.fk_get_launch(precision)
    try:
        F.fk_set_launch(precision, 64, 1, 32)       # 256 wavefronts: every batch below fills their lanes
        for kind in (0, 1):
            kinds = [kind] * len(probs)
            _, ws, PB, _ = F.solve_batch(probs, kinds)
            cover = [F.batch_path_samples(ws, PB, m) for m in range(len(probs))]
            _, ws, PB, _ = F.solve_batch(probs + [other], kinds + [0])
            for m, name in enumerate(FORMS):
                say("kind", kind, "precision", precision, "levels", levels, name)
                v, s = F.batch_path_samples(ws, PB, m)
                assert s.tobytes() == cover[m][1].tobytes(), name
                assert v.tobytes() == cover[m][0].tobytes(), name
            # alone, in a single-problem launch
            for m in (1, 4, 6):
                st, ws1, P = F.solve(probs[m], kind)
                v, s = F.path_samples(ws1, kind, 2, P.params)
                assert s.tobytes() == cover[m][1].tobytes() and v.tobytes() == cover[m][0].tobytes(), m
    finally:
        F.fk_set_launch_dict(precision, keep)


def test_shared_source_of_two_boxes():
    """One grid under a box that it covers and a smaller one: the walk kernel reads one source for both problems."""
    from paper_1709_07469_amd import fkgrav as F
    for precision in (W.PREC_F64, W.PREC_MIXED_F64ACC):
        a = FORMS["general spacings"]().replace(precision=precision)
        b = a.replace(box_lo=np.full(3, -0.8), box_hi=np.full(3, 0.9), stations=a.stations[:1] * 0.5, problem_id=1)
        PB = F.PreparedBatch([a, b, a], [0, 1, 1])
        for q in PB.problems:                       # the same device grid in all: a shared source
            q.source.rho = PB.problems[0].source.rho
        _, ws, _, _ = F.solve_batch(None, None, prepared=PB)
        for m, (p, kind) in enumerate(((a, 0), (b, 1), (a, 1))):
            _, ws1, P = F.solve(p, kind)
            v, s = F.path_samples(ws1, kind, p.n_stations, P.params)
            bv, bs = F.batch_path_samples(ws, PB, m)
            assert s.tobytes() == bs.tobytes() and v.tobytes() == bv.tobytes(), (precision, m)
