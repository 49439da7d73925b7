"""GPU: a launch's wavefronts take their first run of tasks by their place in
the launch, the claim counters the rest.  Around the sizes where the runs cover
the tasks, whatever the stripes, every walk must run once: the records equal,
bit for bit, those of a launch of many more walks."""
import functools

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


def _problem(n):
    pr = W.cfg1(n, precision=W.PREC_MIXED_F64ACC)
    return pr.replace(stations=pr.stations[:1], dt=0.05, max_steps=400)


def _waves(block):
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count * block // 64


@functools.lru_cache(maxsize=None)
def _all(block):
    """More walks than any case needs, from a launch of stripes 1."""
    _, v, s = gpu_solve(_problem(_waves(block) * 64 * 2 + 7), 0)
    return v[0], s[0]


@pytest.mark.parametrize("block", [64, 192, 256])
@pytest.mark.parametrize("stripes", [1, 3, 8, 32])
def test_every_task_runs_once(stripes, block):
    from paper_1709_07469_amd import fkgrav as F
    prec = W.PREC_MIXED_F64ACC
    fv, fs = _all(block)
    w = _waves(block)
    keep = F.fk_get_launch(prec)
    try:
        F.fk_set_launch(prec, block, 1, 32, stripes=stripes)
        for n in (2, 5, 33, w - 1, w + 1, 7 * w + 3, 63 * w, 63 * w + 1, 64 * w - 1, 64 * w, 64 * w + 1,
                  64 * w + 700, 128 * w + 7):
            say("block", block, "stripes", stripes, "walks", n)
            _, v, s = gpu_solve(_problem(n), 0)
            assert v[0].tobytes() == fv[:n].tobytes() and s[0].tobytes() == fs[:n].tobytes(), n
            pr = _problem(n)
            res, ws, PB, _ = F.solve_batch([pr, pr.replace(problem_id=3)], [0, 0])
            bv, bs = F.batch_path_samples(ws, PB, 0)
            assert bv.tobytes() == fv[:n].tobytes() and bs.tobytes() == fs[:n].tobytes(), n
    finally:
        F.fk_set_launch_dict(prec, keep)
