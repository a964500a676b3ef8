"""Sampling under a raised facet threshold (area_eps): every point takes the nearest particle's value and
id exactly, also where the facet lists of two cells overlap because one of them lacks their common
facet, in cells of at most 64 vertices and of more."""
import numpy as np
import pytest

from test_gpu_grid_threshold import _clump, _retried

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,sub", [((30, 30, 30), 1), ((10, 10, 11), 3)])
@pytest.mark.parametrize("eps", [1e-12, 1e-3, 1e-1])
def test_sample(vt, torch_cuda, oracle, eps, dims, sub):
    p = _clump(3, 300, 1200, 0.1)
    n = len(p)
    val = np.random.default_rng(13).uniform(0.5, 2.0, n)
    ctx = vt.Context().vt_build(torch_cuda.from_numpy(p).cuda(), vt.whole_box(n, 0.0, 1.0), area_eps=eps)
    assert len(_retried(ctx.vt_cells())) >= 1
    g, near = ctx.vt_grid_sample(torch_cuda.from_numpy(val).cuda(), dims, sub=sub, nearest=True)
    assert ctx.vt_query()[0] == 0
    gref, nref = oracle.grid_sample(p, 0.0, 1.0, val, dims, sub=sub, chunk=1024)
    assert np.array_equal(near.cpu().numpy(), nref)
    assert np.array_equal(g.cpu().numpy(), gref)


def test_coincident_particles(vt, torch_cuda, oracle):
    # reported as an error of the build, but their common cell's points still go to the smaller id
    rng = np.random.default_rng(17)
    p = rng.random((1500, 3))
    p = np.concatenate([p, p[rng.permutation(1500)[:300]]])[rng.permutation(1800)]
    val = rng.uniform(0.5, 2.0, len(p))
    ctx = vt.Context().vt_build(torch_cuda.from_numpy(p).cuda(), vt.whole_box(len(p), 0.0, 1.0))
    assert ctx.vt_query()[0] == 4
    _, near = ctx.vt_grid_sample(torch_cuda.from_numpy(val).cuda(), (30, 30, 30), nearest=True)
    assert np.array_equal(near.cpu().numpy(), oracle.grid_sample(p, 0.0, 1.0, val, (30, 30, 30), chunk=1024)[1])
