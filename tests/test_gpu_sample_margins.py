"""Sampling where rounding decides: points on the bisector of two particles whose separations are
rounded in units of the period (small cells astride a face of the box, seen through the wrap), and
boxes far from the origin, where the points' own coordinates are rounded in coarse units.  The id is
the one of the brute-force reference's own FP64 distances, ties to the smaller id."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _nearest(p, lo, L, q):
    e = p[None] - q[:, None]
    e = e - L * np.rint(e / L)
    d2 = e[..., 0] * e[..., 0] + e[..., 1] * e[..., 1] + e[..., 2] * e[..., 2]
    return np.argmin(d2, axis=1)


@pytest.mark.parametrize("axis", [0, 2])
@pytest.mark.parametrize("scale", [3e-6, 1e-5, 1e-4])
def test_astride_a_face(vt, torch_cuda, scale, axis):
    rng = np.random.default_rng(31)
    dims = [8, 8, 8]
    dims[axis] = int(0.2 / scale)
    jk = np.stack(np.meshgrid(*[np.arange(1 if a == axis else 8) for a in range(3)], indexing="ij"), -1).reshape(-1, 3)
    q = 0.0 + (jk + 0.5) * (1.0 / np.array(dims))
    u = rng.standard_normal((len(q), 30, 3))
    u /= np.linalg.norm(u, axis=2)[:, :, None]
    shell = (q[:, None] + 8.0 * scale * u * (1.0 + 0.2 * rng.random((len(q), 30, 1)))).reshape(-1, 3)
    a = np.zeros((len(q), 3))
    a[:, axis] = scale * (3.0 + rng.random(len(q)))   # beyond the point's 2.5 scale from the face
    side = np.concatenate([q + a, q - a])
    background = rng.random((3000, 3))
    background = background[(np.abs(background[:, axis] - 0.5) < 0.499)]
    p = np.mod(np.concatenate([side, shell, background]), 1.0)
    p = np.ascontiguousarray(p[rng.permutation(len(p))])
    ctx = vt.Context().vt_build(torch_cuda.from_numpy(p).cuda(), vt.whole_box(len(p), 0.0, 1.0))
    val = torch_cuda.arange(len(p), dtype=torch_cuda.float64, device="cuda")
    _, near = ctx.vt_grid_sample(val, dims, nearest=True)
    assert ctx.vt_query()[0] == 0
    got = near.cpu().numpy()[tuple(jk.T)]
    assert np.array_equal(got, _nearest(p, 0.0, 1.0, q))


@pytest.mark.parametrize("lo", [0.0, 1e5, 1e7])
def test_far_from_the_origin(vt, torch_cuda, lo):
    rng = np.random.default_rng(32)
    dims = (8, 8, 500)
    ii = np.unique(np.stack([rng.integers(0, d, 300) for d in dims], -1), axis=0)
    h = 1.0 / np.array(dims)
    q = lo + (ii + 0.5) * h
    ulp = 2.0 ** -29
    a = np.zeros((len(q), 3))
    a[:, 2] = ulp * rng.integers(1 << 16, 1 << 18, len(q))
    jitter = ulp * rng.integers(-(1 << 22), 1 << 22, (len(q), 3))
    jitter[:, 2] = 0.0
    background = lo + ulp * rng.integers(0, 1 << 29, (2000, 3))
    far = np.ones(len(background), bool)
    for x in q:
        e = background - x
        far &= np.linalg.norm(e - np.rint(e), axis=1) > 0.03
    p = np.concatenate([q + jitter + a, q + jitter - a, background[far]])
    p = np.ascontiguousarray(p[rng.permutation(len(p))])
    ctx = vt.Context().vt_build(torch_cuda.from_numpy(p).cuda(), vt.whole_box(len(p), lo, lo + 1.0))
    val = torch_cuda.arange(len(p), dtype=torch_cuda.float64, device="cuda")
    _, near = ctx.vt_grid_sample(val, dims, nearest=True)
    assert ctx.vt_query()[0] == 0
    got = near.cpu().numpy()[tuple(ii.T)]
    assert np.array_equal(got, _nearest(p, lo, 1.0, q))
