"""The deposit on axes that are fine in x, where a face's column of full voxels is added by the whole
wavefront: columns shorter and longer than a wavefront, in the cell's box in LDS and beyond it, few and
many faces at once, shared and walls.  Tolerance: the shared-face tests', and per axis voxel the
rounding of a plane's place, 1e-16 of the axis (5e-13 of a voxel at 4000)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(60, 2, 2), (250, 1, 1), (300, 9, 2), (4000, 1, 2), (1500, 6, 5)])
@pytest.mark.parametrize("periodic", [True, False])
@pytest.mark.parametrize("n", [400, 1500])
def test_long_columns(vt, torch_cuda, oracle, n, periodic, dims):
    rng = np.random.default_rng(n)
    p = rng.random((n, 3))
    p[: n // 3] = 0.3 + 0.05 * p[: n // 3]
    val = rng.uniform(-1.0, 2.0, n)
    val[rng.random(n) < 0.1] = 0.0
    ctx = vt.Context().vt_build(torch_cuda.from_numpy(p).cuda(), vt.whole_box(n, 0.0, 1.0, periodic=periodic))
    assert ctx.vt_query()[0] == 0
    vmax = float(ctx.vt_cells().volume.max())
    g = ctx.vt_grid_deposit(torch_cuda.from_numpy(val).cuda(), dims).cpu().numpy()
    assert ctx.vt_query()[0] == 0
    ref = oracle.grid(p, 0.0, 1.0, periodic, val, dims)
    tol = 1e-11 * np.abs(val).max() * max(1.0, vmax * np.prod(dims))
    assert np.max(np.abs(g - ref)) <= tol
