"""Sampling by rows at its edges: axes with one or a few points, rows longer than a wavefront, far
fewer points than cells and far more, cells of very different sizes, points on bisectors (a lattice
whose points fall on faces, edges and corners) and several points per voxel.  Values and ids are
copies and must equal the brute-force reference's exactly."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _check(vt, torch_cuda, oracle, p, dims, sub):
    n = len(p)
    val = np.random.default_rng(91).uniform(0.5, 2.0, n)
    ctx = vt.Context().vt_build(torch_cuda.from_numpy(p).cuda(), vt.whole_box(n, 0.0, 1.0))
    g, near = ctx.vt_grid_sample(torch_cuda.from_numpy(val).cuda(), dims, sub=sub, nearest=True)
    assert ctx.vt_query()[0] == 0
    gref, nref = oracle.grid_sample(p, 0.0, 1.0, val, dims, sub=sub, chunk=1024)
    assert np.array_equal(near.cpu().numpy(), nref)
    assert np.array_equal(g.cpu().numpy(), gref)


@pytest.mark.parametrize("dims,sub", [((1, 1, 1), 1), ((1, 1, 1), 3), ((2, 3, 1), 1), ((1, 5, 200), 1), ((3, 2, 67), 4),
                                      ((64, 5, 7), 1), ((40, 36, 44), 1), ((5, 6, 4), 7)])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_shapes(vt, torch_cuda, oracle, dims, sub, dtype):
    rng = np.random.default_rng(92)
    p = np.concatenate([0.4 + 0.01 * rng.normal(size=(900, 3)), rng.random((1600, 3))]).astype(dtype)
    _check(vt, torch_cuda, oracle, np.ascontiguousarray(p), dims, sub)


@pytest.mark.parametrize("dims,sub", [((8, 8, 8), 1), ((16, 16, 16), 1), ((8, 4, 16), 2), ((24, 8, 8), 1)])
def test_points_on_faces(vt, torch_cuda, oracle, dims, sub):
    c = np.arange(8) / 8.0
    p = np.stack(np.meshgrid(c, c, c, indexing="ij"), -1).reshape(-1, 3)
    _check(vt, torch_cuda, oracle, np.ascontiguousarray(p[np.random.default_rng(93).permutation(len(p))]), dims, sub)
