"""GPU: the sizes up to which a grid takes the covering lookup: layers below 2^24
voxels (24-bit products) and grids below 2^30 (32-bit byte addresses, up to
4 GiB less a layer of an FP32 grid), grids at addresses of the least alignment,
and an axis of the greatest length.  On both sides of each limit the route is
read from the profiler, and every walk's record must be that of the general loop
(the same problem in a batch with one whose grid does not cover its box), bit for
bit.  Densities are made on the GPU, from a hash of the voxel's index, so that a
wrong address shows."""
import numpy as np
import pytest

from paper_1709_07469_amd import workloads as W
from gpu_helpers import say
from kernel_names import loops, walk_kernels
from test_gpu_covering_grids import _grid

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _hashed(voxels, levels, skip):
    """A device grid of that many voxels, `skip` elements into its allocation."""
    import torch
    out = torch.empty(voxels + skip, dtype=torch.uint8 if levels else torch.float32, device="cuda")
    for a in range(0, voxels, 1 << 27):
        i = torch.arange(a, min(voxels, a + (1 << 27)), device="cuda")
        h = (((i * 2654435761) & 0xFFFFFFFF) >> 24) ^ ((i >> 20) & 255)      # 0 .. 255
        out[skip + a:skip + a + len(i)] = h if levels else h.to(torch.float32) - 100.5
    return out[skip:]


CASES = [("just below 2^30 voxels", (1024, 1024, 1023), 0, True), ("2^30 voxels", (1024, 1024, 1024), 0, False),
         ("layers just below 2^24", (4096, 4095, 3), 0, True), ("layers of 2^24", (4096, 4096, 3), 0, False),
         ("an axis of 2^24 - 1", (16777215, 1, 1), 0, True), ("unaligned", (37, 41, 29), 1, True)]


@pytest.mark.parametrize("levels", [False, True])
@pytest.mark.parametrize("name, n, skip, covers", CASES, ids=[c[0] for c in CASES])
def test_covering_lookup_at_the_sizes_it_is_limited_to(name, n, skip, covers, levels):
    import torch
    from paper_1709_07469_amd import fkgrav as F
    rho = _hashed(int(np.prod(n)), levels, skip)
    table = torch.arange(256, dtype=torch.float32, device="cuda") - 100.5
    small = (1, 1, 1)

    def at_size(source):
        source.n[:] = n
        source.spacing[:] = [2.0 / k for k in n]
        if levels:
            source.rho_index, source.rho_levels = rho.data_ptr(), table.data_ptr()
        else:
            source.rho = rho.data_ptr()

    plain = 12 if levels else 4
    for precision in (W.PREC_F64, W.PREC_MIXED_F64ACC):
        p = _grid(small, (-1, -1, -1), (2, 2, 2)).replace(precision=precision, grid_levels=levels,
                                                          bc_kind=W.BC_ZERO, bc_data=np.zeros(0))
        other = _grid((16, 16, 16), (-1, -1, -1), (1 / 16,) * 3).replace(precision=precision, grid_levels=levels,
                                                                         problem_id=99, paths_per_station=64)
        keep = F.fk_get_launch(precision)
        try:
            F.fk_set_launch(precision, 64, 1, 32)   # a wavefront a compute unit: lanes filled, so not a capped launch
            say(name, "precision", precision, "levels", levels)
            P = F.Prepared(p)
            at_size(P.source)
            (_, ws, _), ks = walk_kernels(lambda: F.solve(p, 0, prepared=P))
            assert loops(ks) == {plain + (16 if covers else 0)}
            v, s = F.path_samples(ws, 0, p.n_stations, P.params)
            PB = F.PreparedBatch([p, other], [0, 0])
            at_size(PB.problems[0].source)
            (_, ws, _, _), ks = walk_kernels(lambda: F.solve_batch(None, None, prepared=PB))
            assert loops(ks) == {plain}
            bv, bs = F.batch_path_samples(ws, PB, 0)
            assert s.tobytes() == bs.tobytes() and v.tobytes() == bv.tobytes()
            assert len(np.unique(v)) > 500          # zero data: only the densities differ between the walks
        finally:
            F.fk_set_launch_dict(precision, keep)
