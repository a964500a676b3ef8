"""Sampling several points a voxel with about as many points as cells, on both sides of the rule that
chooses tiles of points (powers of two: 65536 cells and points, eight points a cell; other sizes:
300000 cells; twice as fine along one axis as along another): evenly spread particles, tiles cut off by
the grid's end, a clump that leaves the points to the cells (one that shows in the
counts of Morton cells, and a tight one of a few hundred particles among many that does not), and a
lattice whose points have eight nearest particles.  Values are the particles' indices, whose sums over
a voxel are exact, and ids come from a k-d tree, so the averages are equal wherever no other particle
is as near up to rounding."""
import numpy as np
import pytest
from scipy.spatial import cKDTree

pytestmark = pytest.mark.gpu


def _points(dims, sub):
    ax = [((np.arange(d)[:, None] + (np.arange(sub) + 0.5) / sub) / d).reshape(-1) for d in dims]
    return np.stack(np.meshgrid(*ax, indexing="ij"), -1)


def _mean(ids, dims, sub):
    nx, ny, nz = dims
    return ids.reshape(nx, sub, ny, sub, nz, sub).transpose(0, 2, 4, 1, 3, 5).reshape(nx, ny, nz, -1).mean(-1)


def _sample(vt, torch_cuda, p, dims, sub):
    ctx = vt.Context().vt_build(torch_cuda.from_numpy(p).cuda(), vt.whole_box(len(p), 0.0, 1.0))
    val = torch_cuda.arange(len(p), dtype=torch_cuda.float64, device="cuda")
    got = [ctx.vt_grid_sample(val, dims, sub=sub).cpu().numpy() for _ in range(2)]
    assert ctx.vt_query()[0] == 0
    assert np.array_equal(got[0], got[1])
    return got[0]


@pytest.mark.parametrize("kind", ["even", "clump", "tight"])
@pytest.mark.parametrize("n,dims,sub", [(65535, (32, 16, 16), 2), (65536, (32, 16, 16), 2), (65536, (16, 16, 15), 2),
                                        (70001, (16, 16, 8), 4), (32769, (32, 32, 32), 2), (299999, (22, 23, 24), 2),
                                        (300000, (22, 23, 24), 2), (300000, (15, 21, 13), 3), (310000, (44, 22, 23), 2),
                                        (310000, (45, 22, 23), 2)])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_against_kdtree(vt, torch_cuda, n, dims, sub, kind, dtype):
    rng = np.random.default_rng(n)
    p = rng.random((n, 3))
    if kind == "clump":
        p[: n // 3] = 0.4 + 0.03 * rng.standard_normal((n // 3, 3))
    elif kind == "tight":
        p[:400] = 0.7 + 0.002 * rng.standard_normal((400, 3))
    p = p.astype(dtype)
    g = _sample(vt, torch_cuda, p, dims, sub)
    q = _points(dims, sub)
    d, j = cKDTree(p.astype(np.float64), boxsize=1.0).query(q.reshape(-1, 3), k=2)
    clear = d[:, 1] - d[:, 0] > 1e-12
    whole = _mean(clear.astype(np.float64), dims, sub) == 1.0
    assert whole.mean() > 0.999
    assert np.array_equal(g[whole], _mean(j[:, 0].astype(np.float64), dims, sub)[whole])


def test_lattice_ties(vt, torch_cuda):
    m, dims, sub = 64, (32, 32, 32), 2
    c = np.arange(m) / m
    ids = np.random.default_rng(5).permutation(m ** 3).reshape(m, m, m)
    p = np.empty((m ** 3, 3))
    p[ids.reshape(-1)] = np.stack(np.meshgrid(c, c, c, indexing="ij"), -1).reshape(-1, 3)
    g = _sample(vt, torch_cuda, p, dims, sub)
    low = ids
    for a in range(3):
        low = np.minimum(low, np.roll(low, -1, axis=a))   # the eight corners around each point
    assert np.array_equal(g, _mean(low.astype(np.float64), dims, sub))
