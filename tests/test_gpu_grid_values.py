"""The deposit of a field with a value that is not a number or not finite (a masked particle): the
voxels that its cell covers take it, and every voxel outside the cell's bounding box is untouched by
it.  Tolerance of the others: the shared-face tests'."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("n,dims", [(400, (20, 22, 18)), (3000, (30, 28, 33))])
def test_masked_cells(vt, torch_cuda, oracle, n, dims, bad):
    rng = np.random.default_rng(n)
    p = rng.random((n, 3))
    val = rng.uniform(0.5, 2.0, n)
    masked = [5, 171, 390]
    t = torch_cuda.from_numpy(p).cuda()
    ctx = vt.Context().vt_build(t, vt.whole_box(n, 0.0, 1.0))
    vmax = float(ctx.vt_cells().volume.max())
    x = val.copy()
    x[masked] = bad
    g = ctx.vt_grid_deposit(torch_cuda.from_numpy(x).cuda(), dims).cpu().numpy()
    assert ctx.vt_query()[0] == 0
    covered = np.zeros(dims, bool)
    near = np.zeros(dims, bool)
    for i in masked:
        covered |= oracle.grid(p, 0.0, 1.0, True, np.eye(1, n, i)[0], dims, query=[i]) > 1e-6
        verts = oracle.structure(p, 0.0, 1.0, i)[0]
        rng_ = [np.arange(int(np.floor(verts[:, a].min() * d - 1e-9)), int(np.floor(verts[:, a].max() * d + 1e-9)) + 1) % d
                for a, d in enumerate(dims)]
        near[np.ix_(*rng_)] = True
    assert covered.any() and not (covered & ~near).any()
    got = g[covered]
    assert np.isnan(got).all() if np.isnan(bad) else (got == bad).all()
    x[masked] = 0.0
    ref = oracle.grid(p, 0.0, 1.0, True, x, dims)
    tol = 1e-11 * val.max() * max(1.0, vmax * np.prod(dims))
    assert np.max(np.abs(g - ref)[~near]) <= tol
