"""GPU: covering grids in batches whose problems share one grid (u and g_z of one
voxel model, and the same model under another box), in launches that fill their
lanes: the walk kernel reads the one source, with the bounds and the margin that
hold for all the problems.  Every walk's record must be that of the general loop
(the batch with a problem whose box the grid does not cover) and of the single
solve, bit for bit.  Boxes that leave each other too little of the common bounds
take the general loop."""
import numpy as np
import pytest

from paper_1709_07469_amd import workloads as W
from gpu_helpers import say
from kernel_names import loops, walk_kernels
from test_gpu_covering_grids import FORMS

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _one_grid(probs, kinds):
    """The batch with the first problem's device grid in all: a shared source."""
    from paper_1709_07469_amd import fkgrav as F
    PB = F.PreparedBatch(probs, kinds)
    for q in PB.problems:
        q.source.rho, q.source.rho_index = PB.problems[0].source.rho, PB.problems[0].source.rho_index
        q.source.rho_levels = PB.problems[0].source.rho_levels
    (_, ws, _, _), ks = walk_kernels(lambda: F.solve_batch(None, None, prepared=PB))
    assert [name for name, _ in ks] == ["batch_walk_kernel"] and ks[0][1][3] is True     # a shared source
    return [F.batch_path_samples(ws, PB, m) for m in range(len(probs))], ks


@pytest.mark.parametrize("levels", [False, True])
@pytest.mark.parametrize("precision", [W.PREC_F64, W.PREC_MIXED_F64ACC, W.PREC_MIXED_KAHAN])
@pytest.mark.parametrize("form", ["powers of two", "general spacings", "beyond the box", "bodies beside"])
def test_one_covering_grid_for_all_problems(form, precision, levels):
    from paper_1709_07469_amd import fkgrav as F
    a = FORMS[form]().replace(precision=precision, grid_levels=levels)
    b = a.replace(box_hi=np.array([1.0, 0.997, 1.0]), stations=a.stations[:1] * 0.5, problem_id=2)
    c = a.replace(box_lo=np.array([-0.998, -1.0, -1.0]), dt=0.4 * a.dt, problem_id=3)
    wide = a.replace(box_lo=np.full(3, -2.0), box_hi=np.full(3, 2.0), problem_id=9, paths_per_station=64)
    small = a.replace(box_lo=np.full(3, -0.8), box_hi=np.full(3, 0.9), stations=a.stations[:1] * 0.5, problem_id=4)
    seeds = a.replace(seed=5, problem_id=1)
    plain, cover = (12, 28) if levels else (4, 20)
    keep = F.fk_get_launch(precision)
    try:
        F.fk_set_launch(precision, 64, 1, 32)       # a wavefront a compute unit: lanes filled, so not a capped launch
        for probs, kinds, loop in (([a, a.replace(problem_id=1)], [0, 1], cover),     # u and g_z of a model
                                   ([a, seeds], [0, 1], cover),                       # a key each
                                   ([a, b, c], [1, 0, 1], cover),                     # three boxes
                                   ([b, small, a], [0, 1, 1], plain)):                # too little in common
            say(form, "precision", precision, "levels", levels, "loop", loop)
            got, ks = _one_grid(probs, kinds)
            assert loops(ks) == {loop}
            general, ks = _one_grid(probs + [wide], kinds + [0])
            assert loops(ks) == {plain}
            for m, (p, kind) in enumerate(zip(probs, kinds)):
                _, ws, P = F.solve(p, kind)
                v, s = F.path_samples(ws, kind, p.n_stations, P.params)
                for bv, bs in (got[m], general[m]):
                    assert s.tobytes() == bs.tobytes() and v.tobytes() == bv.tobytes(), m
    finally:
        F.fk_set_launch_dict(precision, keep)
