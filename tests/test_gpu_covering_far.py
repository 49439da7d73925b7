"""GPU: covering grids so far from the origin that the FP64 lookup's rounding
margin is a visible part of a voxel.  Macro-steps with a point that near a voxel
face take the general lookup instead, hundreds of times in each case here; grids
whose margin exceeds 2^-12 of a voxel take the general loop from the start.
Every walk's record must be that of the general loop, bit for bit (the same
problem in a batch with one whose grid does not cover its box)."""
import numpy as np
import pytest

from paper_1709_07469_amd import workloads as W
from gpu_helpers import MASK, say
from kernel_names import loops, walk_kernels
from test_gpu_covering_grids import _grid

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _far(log2, n, sign):
    """A grid over a box of edge 2 with its origin 2^log2 voxels out on every axis."""
    d = 2.0 / np.asarray(n, float)
    lo = sign * d * 2.0 ** log2
    return _grid(n, lo, d, lo, lo + 2)


def _margin(p):
    x = np.maximum(np.abs(p.box_lo), np.abs(p.box_hi)) + 9 * np.sqrt(p.dt)
    return float(np.max(2.0 ** -51 * ((x + np.abs(p.grid_origin)) / p.grid_spacing + np.array(p.rho.shape[::-1]) + 2)))


@pytest.mark.parametrize("levels", [False, True])
@pytest.mark.parametrize("log2, n, sign", [(35, (33, 29, 27), 1), (36.4, (31, 50, 23), -1), (37.7, (27, 33, 29), 1),
                                           (40, (33, 29, 27), -1)])
def test_far_grids_equal_the_general_loop(log2, n, sign, levels):
    from paper_1709_07469_amd import fkgrav as F
    p = _far(log2, n, sign).replace(grid_levels=levels)
    far = _margin(p) > 2.0 ** -12
    assert far == (log2 == 40)
    other = _grid((16, 16, 16), (-1, -1, -1), (1 / 16,) * 3).replace(grid_levels=levels, problem_id=99,
                                                                     paths_per_station=64)
    keep = F.fk_get_launch(p.precision)
    try:
        F.fk_set_launch(p.precision, 64, 1, 32)     # a wavefront a compute unit: lanes filled, so not a capped launch
        for kind in (0, 1):
            say("origin at 2 ^", log2, "voxels, kind", kind, "levels", levels)
            (_, ws, PB, _), ks = walk_kernels(lambda: F.solve_batch([p, other], [kind, 0]))
            assert loops(ks) == {12 if levels else 4}
            v, s = F.batch_path_samples(ws, PB, 0)
            (_, ws1, P), ks = walk_kernels(lambda: F.solve(p, kind))
            assert loops(ks) == {(12 if levels else 4) + (0 if far else 16)}
            v1, s1 = F.path_samples(ws1, kind, p.n_stations, P.params)
            assert s1.tobytes() == s.tobytes() and v1.tobytes() == v.tobytes()
            q = p.replace(problem_id=3)             # two sources of their own in a batch
            (_, ws2, PB, _), ks = walk_kernels(lambda: F.solve_batch([p, q], [kind, 0]))
            assert loops(ks) == {(12 if levels else 4) + (0 if far else 16)}
            v2, s2 = F.batch_path_samples(ws2, PB, 0)
            assert s2.tobytes() == s.tobytes() and v2.tobytes() == v.tobytes()
            if not far:     # points expected within the margin of a face, on either side of it and on three axes
                assert np.sum(s & MASK, dtype=np.float64) * 6 * _margin(p) > 100
    finally:
        F.fk_set_launch_dict(p.precision, keep)
