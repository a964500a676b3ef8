"""The deposit with each face integrated once for its two cells: cells that take part next to cells
that do not (zero values, buffer particles, cells inside one voxel, walls), values of both signs,
voxels much larger and much smaller than the cells, one cell and few cells per wavefront.

Tolerance per voxel: its value is a sum of signed region integrals, each at most a cell's volume in
voxels times the largest value, with rounding of the order of 1e-16 times a few hundred terms and
their conditioning: 1e-11 of max|value| max(1, V_max / V_voxel)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _check(vt, torch_cuda, oracle, p, periodic, val, dims, items=None, ids=None):
    t = torch_cuda.from_numpy(p).cuda()
    n = len(val)
    ctx = vt.Context().vt_build(t, items or vt.whole_box(len(p), 0.0, 1.0, periodic=periodic))
    vmax = float(ctx.vt_cells().volume.max())
    g = ctx.vt_grid_deposit(torch_cuda.from_numpy(val).cuda(), dims).cpu().numpy()
    assert ctx.vt_query()[0] == 0
    full = np.zeros(len(p))
    full[:n] = val
    ref = oracle.grid(p, 0.0, 1.0, periodic, full, dims, query=np.arange(n))
    tol = 1e-11 * np.abs(val).max() * max(1.0, vmax * np.prod(dims))
    assert np.max(np.abs(g - ref)) <= tol


@pytest.mark.parametrize("dims", [(1, 1, 1), (3, 5, 2), (11, 1, 40), (40, 33, 27)])
@pytest.mark.parametrize("periodic", [True, False])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_mixed_values(vt, torch_cuda, oracle, dims, periodic, dtype):
    rng = np.random.default_rng(71)
    p = rng.random((2000, 3))
    p[:700] = 0.5 + 0.03 * rng.normal(size=(700, 3))   # small cells next to large ones
    p = np.clip(p, 1e-6, 1 - 1e-6).astype(dtype)
    val = rng.uniform(-1.0, 2.0, len(p))
    val[rng.random(len(p)) < 0.3] = 0.0
    _check(vt, torch_cuda, oracle, p.astype(dtype), periodic, val, dims)


def test_buffer_particles(vt, torch_cuda, oracle):
    rng = np.random.default_rng(72)
    p = rng.random((1500, 3))
    items = [dict(offset=0, n_owned=900, n_ghost=600, periodic=False, lo=np.zeros(3), hi=np.ones(3), walls=0)]
    _check(vt, torch_cuda, oracle, p, False, rng.uniform(0.5, 2.0, 900), (9, 14, 12), items=items)


@pytest.mark.parametrize("n", [600, 9000, 20011])
def test_cells_per_turn(vt, torch_cuda, oracle, n):
    rng = np.random.default_rng(73)
    _check(vt, torch_cuda, oracle, rng.random((n, 3)), True, rng.uniform(0.5, 2.0, n), (12, 10, 14))
