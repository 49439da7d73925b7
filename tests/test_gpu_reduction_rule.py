"""GPU: when a reduction with prism data forms its samples in a pass of its own.
Several blocks then share a pair; with only two blocks for each (more than a third
of 8 blocks per compute unit in pairs) the pass costs more than it saves, and
with fewer than 8 walks a lane as well.  The kernels that ran are read from the
profiler; whichever form a solve takes, its stations' results are the same, bit
for bit (a station's walks do not depend on how many stations there are)."""
import re

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


def _solve(stations, n, kind):
    """Statistics, and the passes the reduction took (0: whole, 1: samples, 2: from samples)."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    from paper_1709_07469_amd import fkgrav as F
    p = W.cfg2(n, precision=W.PREC_MIXED_F64ACC)
    p = p.replace(dt=2500.0, stations=np.tile(p.stations, (stations // p.n_stations + 1, 1))[:stations])
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        st, _, _ = F.solve(p, kind)
        torch.cuda.synchronize()
    found = [re.search(r"chunk_kernel<(\d)>", e.name) for e in prof.events()]
    return st, sorted(int(m.group(1)) for m in found if m)


@pytest.mark.parametrize("kind, n, passes", [(0, 1792, 1), (0, 1793, 2), (1, 896, 1), (1, 897, 2), (1, 4096, 2)])
def test_two_passes_need_three_blocks_a_pair_and_eight_walks_a_lane(kind, n, passes):
    import torch
    full = 8 * torch.cuda.get_device_properties(0).multi_processor_count
    few = full // 3                                        # 3 blocks a pair; with one pair more, 2
    say("kind", kind, "walks a pair", n * (kind + 1), "pairs", few)
    a, ran = _solve(few, n, kind)
    assert ran == ([1, 2] if passes == 2 else [0])
    b, ran = _solve(few + 1, n, kind)
    assert ran == [0]
    assert a.tobytes() == b[:few].tobytes()
