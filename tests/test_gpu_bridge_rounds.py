"""GPU: shared drain rounds gather the steps that need the bridge test before
they make it.  With no step near a face, some, and every one (several passes of
tests), and with caps among the stops, every walk's record must equal, bit for
bit, that of a launch that fills its wavefronts."""
import numpy as np
import pytest

from paper_1709_07469_amd import workloads as W
from gpu_helpers import gpu_solve, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _problem(domain, dt, n, precision):
    if domain == "box":
        pr = W.cfg3(n, precision=precision, n=32)
        return pr.replace(stations=pr.stations[100:101], dt=dt, exit_rule=W.EXIT_BRIDGE, max_steps=100)
    pr = W.paper_ball(stations=np.array([[0.05, 0.05, 0.2]]), dt_paper=100 * dt, paths_per_station=n,
                      precision=precision)
    return pr.replace(exit_rule=W.EXIT_BRIDGE, max_steps=100)


@pytest.mark.parametrize("precision", [W.PREC_F64, W.PREC_MIXED_F64ACC, W.PREC_MIXED_KAHAN])
@pytest.mark.parametrize("dt", [1e-5, 2e-3, 5e-2])
@pytest.mark.parametrize("domain", ["box", "ball"])
def test_gathered_bridge_tests_record_the_same_walks(domain, dt, precision):
    import torch
    from paper_1709_07469_amd import fkgrav as F
    waves = torch.cuda.get_device_properties(0).multi_processor_count
    keep = F.fk_get_launch(precision)
    try:
        F.fk_set_launch(precision, 64, 1, 32)
        _, fv, fs = gpu_solve(_problem(domain, dt, waves * 66, precision), 0)
        for share in (1, 2, 5, 21):
            n = waves * share
            say(domain, "dt", dt, "precision", precision, "walks per wavefront", share)
            _, v, s = gpu_solve(_problem(domain, dt, n, precision), 0)
            assert v[0].tobytes() == fv[0, :n].tobytes() and s[0].tobytes() == fs[0, :n].tobytes(), share
    finally:
        F.fk_set_launch_dict(precision, keep)
