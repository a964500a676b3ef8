"""The structure of cells of more and fewer than 64 vertices some of whose faces are slivers of rounding width:
neighbours placed so that their planes pass through an edge of a cell (or a gap inside it), with a
facet threshold low enough to keep whatever rounding leaves of such faces.  Clipped again in another
order the cell need not close: it is then left empty and reported.  Otherwise its loops are there and
use every vertex."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def sliver_world(oracle, seed, n_shell=80, n_sliver=40):
    rng = np.random.default_rng(seed)
    u = rng.standard_normal((n_shell, 3))
    u /= np.linalg.norm(u, axis=1)[:, None]
    c = np.full(3, 0.5)
    shell = c + (0.2 + 0.004 * rng.random((n_shell, 1))) * u
    far = rng.random((400, 3))
    far = far[np.linalg.norm(far - c, axis=1) > 0.27]
    p = np.concatenate([[c], shell, far])
    verts, faces = oracle.structure(p, 0.0, 1.0, 0)
    verts = verts - c
    edges = {}
    for j, loop in faces:
        for a, b in zip(loop, np.roll(loop, -1)):
            edges.setdefault((min(a, b), max(a, b)), []).append(j)
    extra = []
    for (a, b), (j, k) in sorted(edges.items()):
        d = verts[b] - verts[a]
        if np.linalg.norm(d) < 0.01:
            continue
        q = verts[a] - d * (verts[a] @ d) / (d @ d)   # the edge's line at its nearest to the seed
        w = np.linalg.lstsq(np.stack([p[j] - c, p[k] - c], 1), q, rcond=None)[0]
        if w.min() > 0.05:   # the plane through the edge lies between its two faces
            extra.append(c + 2.0 * q)
    extra = np.array(extra)[rng.permutation(len(extra))[:n_sliver]]
    return np.concatenate([[c], extra, shell, far]), len(extra)


@pytest.mark.parametrize("eps", [1e-30, 1e-12])
@pytest.mark.parametrize("gap", [0.0, 1e-15, 3e-15, 1e-10])
@pytest.mark.parametrize("seed", range(5))
def test_slivers(vt, torch_cuda, oracle, seed, gap, eps):
    p, n_sliver = sliver_world(oracle, seed)
    own = slice(1, 1 + n_sliver)
    p[own] = p[0] + (p[own] - p[0]) * (1.0 - gap)
    n = len(p)
    ctx = vt.Context().vt_build(torch_cuda.from_numpy(p).cuda(), vt.whole_box(n, 0.0, 1.0), want_faces=True, area_eps=eps)
    cells = ctx.vt_cells()
    assert int(cells.status[0]) & 2
    _check_row(ctx, 0)


def _check_row(ctx, i):
    s = ctx.vt_structure()
    code = ctx.vt_query()[0]
    vo, fo, lo = (t.cpu().numpy() for t in (s.vert_off, s.face_off, s.loop_off))
    if vo[i + 1] == vo[i]:
        assert code == 8 and fo[i + 1] == fo[i]
        return
    lv = s.loop_vert.cpu().numpy()
    loops = [lv[lo[f]:lo[f + 1]] for f in range(fo[i], fo[i + 1])]
    assert min(len(x) for x in loops) >= 3
    assert np.array_equal(np.unique(np.concatenate(loops)), np.arange(vo[i + 1] - vo[i]))


@pytest.mark.parametrize("gap", [0.0, 2e-16, 5e-16])
@pytest.mark.parametrize("n_shell,n_sliver,seed", [(18, 8, 8), (14, 10, 20), (18, 8, 7), (14, 10, 3)])
def test_slivers_of_small_cells(vt, torch_cuda, oracle, n_shell, n_sliver, seed, gap):
    p, k = sliver_world(oracle, seed, n_shell, n_sliver)
    p[1:1 + k] = p[0] + (p[1:1 + k] - p[0]) * (1.0 - gap)
    ctx = vt.Context().vt_build(torch_cuda.from_numpy(p).cuda(),
                                vt.whole_box(len(p), 0.0, 1.0, periodic=False, walls=63), want_faces=True, area_eps=1e-30)
    assert ctx.vt_query()[0] == 0
    _check_row(ctx, 0)
