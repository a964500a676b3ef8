"""The deposit of lattices, whose cells' vertices lie on many planes at once: their records hold faces
all of whose edges have length zero, or that are folded to a line, which must add nothing.  Box lengths
with and without rounding in the positions, the cell count an input's symmetry can break.  Tolerance:
the shared-face tests'."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(9, 1, 1), (5, 1, 24), (12, 8, 8), (43, 8, 23), (130, 3, 2)])
@pytest.mark.parametrize("lo,size", [(0.0, 62.5), (100.0, 62.5), (-3.0, 62.5), (0.0, 1.0)])
@pytest.mark.parametrize("m,offset", [(4, 0.0), (4, 0.5), (8, 0.0), (16, 0.5)])
def test_cubic(vt, torch_cuda, oracle, m, offset, lo, size, dims):
    rng = np.random.default_rng(m)
    c = lo + size * (np.arange(m) + offset) / m
    p = np.stack(np.meshgrid(c, c, c, indexing="ij"), -1).reshape(-1, 3)[rng.permutation(m ** 3)]
    val = rng.uniform(0.1, 2.0, len(p))
    for values in (val, np.where(rng.random(len(p)) < 0.5, val, 0.0)):
        ctx = vt.Context().vt_build(torch_cuda.from_numpy(p).cuda(), vt.whole_box(len(p), lo, lo + size))
        assert ctx.vt_query()[0] == 0
        g = ctx.vt_grid_deposit(torch_cuda.from_numpy(values).cuda(), dims).cpu().numpy()
        assert ctx.vt_query()[0] == 0
        ref = oracle.grid(p, lo, lo + size, True, values, dims)
        assert np.max(np.abs(g - ref)) <= 1e-11 * 2.0 * max(1.0, np.prod(dims) / m ** 3)
