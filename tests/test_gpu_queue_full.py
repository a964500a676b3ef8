"""More cells of over 64 vertices than the large clip kernel's queue holds (4096 here): those that find
it full are reported failed, with no volume, no neighbours and no part in the deposit, and the others
are what they are alone.  Each is a seed in a shell of 60 buffer particles; the cells are disjoint and
compared with the oracle's, the deposit's total with theirs (a sum of 4096 cells' exact integrals,
1e-16 each of a few hundred terms: 1e-12)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_dropped_cells(vt, torch_cuda, oracle):
    rng = np.random.default_rng(61)
    g = 17
    c = (np.stack(np.meshgrid(*[np.arange(g)] * 3, indexing="ij"), -1).reshape(-1, 3) + 0.5) / g
    u = rng.standard_normal((60, 3))
    u /= np.linalg.norm(u, axis=1)[:, None]
    shell = 0.3 / g * u * (1.0 + 0.02 * rng.random((60, 1)))
    n = len(c)
    p = np.concatenate([c, (c[:, None, :] + shell).reshape(-1, 3)])
    items = vt.whole_box(n, 0.0, 1.0, periodic=False)
    items[0]["n_ghost"] = len(p) - n
    t = torch_cuda.from_numpy(p).cuda()
    ones = torch_cuda.ones(n, dtype=torch_cuda.float64, device="cuda")
    ctx = vt.Context()
    for _ in range(2):
        ctx.vt_build(t, items)
        assert ctx.vt_query()[0] == 6
        cells = ctx.vt_cells(check=False)
        st, vol = cells.status.cpu().numpy(), cells.volume.cpu().numpy()
        nnb = np.diff(cells.nbr_off.cpu().numpy())
        failed = (st & 4) != 0
        assert failed.sum() == n - 4096
        assert np.all(vol[failed] == 0.0) and np.all(nnb[failed] == 0)
        alone = np.concatenate([c[:1], c[0] + shell])
        ref = oracle.cells(alone, 0.0, 1.0, periodic=False, query=[0])
        assert np.all(nnb[~failed] == ref.nnb[0]) and np.allclose(vol[~failed], ref.volume[0], rtol=1e-12, atol=0)
        grid = ctx.vt_grid_deposit(ones, (40, 23, 31))
        assert abs(float(grid.sum()) / (40 * 23 * 31) - vol.sum()) <= 1e-12 * vol.sum()
