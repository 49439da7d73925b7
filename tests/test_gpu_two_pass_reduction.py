"""GPU: launches with few (station, chunk) pairs and prism data form their
samples in a pass of several blocks per pair before the reduction; launches of
many pairs form them as they reduce.  A station's samples and result must not
depend on which: bit for bit, with capped walks among them, with and without
kept records, alone and in a batch, in stations of one chunk and of two."""
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


@pytest.mark.parametrize("slice_walks", [0, 1 << 15])
@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("paths", [896, 897, 1792, 1793, 8192, 8192 + 700])
def test_samples_of_few_pairs_equal_those_of_many(paths, kind, slice_walks):
    import torch
    from paper_1709_07469_amd import fkgrav as F
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    base = W.cfg2(paths, precision=W.PREC_MIXED_F64ACC)
    pairs = 8 * cus + 1                                   # enough for the one-pass route, in one launch
    many = -(-pairs // (-(-paths // 8192)))
    st = np.repeat(base.stations[40:41], many, axis=0)
    base = base.replace(dt=400.0, max_steps=250, slice_walks=0)
    full, ws, P, *_ = F.solve(base.replace(stations=st), kind)
    fv, fs = F.path_samples(ws, kind, many, P.params)
    few = base.replace(stations=st[:2], slice_walks=slice_walks)
    say("paths", paths, "kind", kind, "slice", slice_walks, "stations", many, "capped", full["n_trunc"][0])
    assert full["n_trunc"][0] > 0
    a, ws, P, *_ = F.solve(few, kind)
    assert a.tobytes() == full[:2].tobytes()
    if slice_walks == 0:
        v, s = F.path_samples(ws, kind, 2, P.params)
        assert v.tobytes() == fv[:2].tobytes() and s.tobytes() == fs[:2].tobytes()
    b, *_ = F.solve_batch([few, few.replace(stations=st[:1])], [kind, kind])
    assert b[0].tobytes() == a.tobytes() and b[1].tobytes() == a[:1].tobytes()
