"""The deposit on an axis of more than 1e9 voxels (9.6 GB of them): a bounded world of cells stacked
along x, all of value 1, which fill every voxel.  A plane's place is rounded to 1e-16 of the world's
length, 1.3e-7 of a voxel at 1.2e9, a few of which make a voxel's error: 1e-6."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_more_than_a_billion_voxels(vt, torch_cuda):
    n, nx = 40000, 1200000000
    rng = np.random.default_rng(5)
    p = np.full((n, 3), 5e-6)
    p[:, 0] = (np.arange(n) + 0.5 + 0.2 * rng.uniform(-1.0, 1.0, n)) / n
    items = [dict(offset=0, n_owned=n, n_ghost=0, periodic=False, lo=np.zeros(3), hi=np.array([1.0, 1e-5, 1e-5]), walls=63)]
    ctx = vt.Context().vt_build(torch_cuda.from_numpy(p).cuda(), items)
    assert ctx.vt_query()[0] == 0
    g = ctx.vt_grid_deposit(torch_cuda.ones(n, dtype=torch_cuda.float64, device="cuda"), (nx, 1, 1))
    assert ctx.vt_query()[0] == 0
    assert float((g - 1.0).abs().max()) <= 1e-6
