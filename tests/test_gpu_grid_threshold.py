"""The deposit under a raised facet threshold (area_eps), next to cells of more than 64 vertices, whose
geometry is kept as their facet list and so lacks the facets below their own threshold.  Every cell
deposits a closed polytope of its own, the true cell, or for such a cell the one its listed facets
bound, so the reference is the sum of both over the cells.  A face integrated once for two cells of
which only one has it would leave the other open.  Tolerance: the shared-face tests'."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _clump(seed, n_uniform=300, n_clump=2500, radius=0.03):
    """A ball of particles in a sparse background: small cells beside large ones of many vertices."""
    rng = np.random.default_rng(seed)
    u = rng.standard_normal((n_clump, 3))
    u /= np.linalg.norm(u, axis=1)[:, None]
    ball = 0.5 + radius * u * rng.random((n_clump, 1)) ** (1 / 3)
    return np.concatenate([rng.random((n_uniform, 3)), ball])


def _retried(cells):
    return np.nonzero(cells.status.cpu().numpy() & 2)[0]


@pytest.mark.parametrize("dims", [(32, 32, 32), (90, 7, 13)])
@pytest.mark.parametrize("eps", [1e-12, 1e-4, 1e-3])
@pytest.mark.parametrize("seed", [1, 2])
def test_deposit(vt, torch_cuda, oracle, seed, eps, dims):
    p = _clump(seed)
    n = len(p)
    ctx = vt.Context().vt_build(torch_cuda.from_numpy(p).cuda(), vt.whole_box(n, 0.0, 1.0), area_eps=eps)
    cells = ctx.vt_cells()
    big = _retried(cells)
    assert len(big) >= 3
    off, ids = cells.nbr_off.cpu().numpy(), cells.nbr_ids.cpu().numpy()
    val = np.random.default_rng(seed + 10).uniform(0.5, 2.0, n)
    g = ctx.vt_grid_deposit(torch_cuda.from_numpy(val).cuda(), dims).cpu().numpy()
    assert ctx.vt_query()[0] == 0
    small = np.setdiff1d(np.arange(n), big)
    ref = oracle.grid(p, 0.0, 1.0, True, np.where(np.isin(np.arange(n), big), 0.0, val), dims, query=small)
    for i in big:
        own = np.concatenate([[i], ids[off[i]:off[i + 1]]])
        ref += oracle.grid(p[own], 0.0, 1.0, True, np.where(own == i, val[i], 0.0), dims, query=[0])
    tol = 1e-11 * val.max() * max(1.0, float(cells.volume.max()) * np.prod(dims))
    assert np.max(np.abs(g - ref)) <= tol
