"""The slab histogram at its other limit: counted in LDS if there are more particles than entries (27
tasks x 6 x 40 here), else in global memory.  Thicknesses equal the oracle's rule exactly."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [50, 6479, 6480, 6481])
@pytest.mark.parametrize("periodic", [True, False])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_thickness(vt, torch_cuda, oracle, n, periodic, dtype):
    p = np.random.default_rng(n).random((n, 3)).astype(dtype)
    thick = vt.Context().vt_decompose(torch_cuda.from_numpy(p).cuda(), 0.0, 1.0, (3, 3, 3), border_factor=1.5,
                                      n_steps=40, periodic=periodic)[0]
    ref = oracle.autoborder(p, 0.0, 1.0, (3, 3, 3), border_factor=1.5, steps=40, periodic=periodic)
    np.testing.assert_allclose(thick, ref, rtol=1e-14, atol=0)
