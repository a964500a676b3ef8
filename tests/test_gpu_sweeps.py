"""Cells whose later shells hold thousands of particles (sparse particles around a smooth-edged clump):
the sweeps' rejection by the box around the vertices and their one-by-one tests of a chunk's few
survivors, in both precisions and away from the origin.  Neighbours equal the oracle's, volumes are
within the FP64 path's 1e-12 and the mixed path's 2e-5."""
import numpy as np
import pytest

from test_gpu_parity import TOL, compare_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("lo,size,dtype", [(0.0, 1.0, np.float64), (-300.0, 100.0, np.float32)])
def test_sparse_cells_around_a_clump(vt, torch_cuda, oracle, precision, lo, size, dtype):
    rng = np.random.default_rng(95)
    clump = 0.5 + 0.03 * rng.standard_normal((6000, 3))
    p = np.concatenate([rng.random((250, 3)), np.clip(clump, 0.01, 0.99)])
    p = (lo + size * p).astype(dtype)
    ctx = vt.Context().vt_build(torch_cuda.from_numpy(p).cuda(), vt.whole_box(len(p), lo, lo + size), precision=precision)
    assert ctx.vt_query()[0] == 0
    cells = ctx.vt_cells()
    ref = oracle.cells(p, lo, lo + size)
    compare_rows(cells, ref, np.arange(len(p)), TOL[precision], "sparse cells")
    assert abs(cells.volume.cpu().numpy().sum() / size ** 3 - 1.0) < 1e-12
