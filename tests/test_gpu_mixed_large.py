"""Large cells in mixed precision with near-parallel planes (pairs of particles a few thousandths to a
few hundred-thousandths apart on the sphere around the seed), whose vertices FP32 cannot place: the
large kernel's FP64 vertices.  Neighbours equal the oracle's in both precisions, volumes are within the
mixed path's 2e-5 and the FP64 path's 1e-12.  (At the smallest gap the pairs' own cells, which the other
kernel computes, have vertices without any FP32 bound: the mixed path reports the box as too small.)"""
import numpy as np
import pytest

from test_gpu_parity import TOL, compare_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gap", [3e-3, 3e-4, 3e-5])
@pytest.mark.parametrize("n", [60, 100])
def test_near_parallel_planes(vt, torch_cuda, oracle, n, gap):
    rng = np.random.default_rng(97)
    u = rng.standard_normal((n, 3))
    u /= np.linalg.norm(u, axis=1)[:, None]
    shell = 0.5 + (0.2 + 0.004 * rng.random((n, 1))) * u
    pair = shell[: n // 3] + gap * rng.standard_normal((n // 3, 3))
    far = rng.random((400, 3))
    far = far[np.linalg.norm(far - 0.5, axis=1) > 0.26]
    p = np.concatenate([[[0.5, 0.5, 0.5]], shell, pair, far])
    t = torch_cuda.from_numpy(p).cuda()
    ref = oracle.cells(p, 0.0, 1.0)
    for precision in (1, 0):
        ctx = vt.Context().vt_build(t, vt.whole_box(len(p), 0.0, 1.0), precision=precision)
        code, _, retried, _ = ctx.vt_query()
        if precision == 1 and gap < 1e-4:
            assert code == 5
            continue
        assert code == 0 and retried >= 1
        compare_rows(ctx.vt_cells(), ref, np.arange(len(p)), TOL[precision], "precision %d" % precision)
