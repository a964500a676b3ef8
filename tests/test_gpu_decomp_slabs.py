"""The slab histogram's two places to count (LDS up to 32768 entries, global memory beyond) at both
sides of the limit, one task, particle counts around a block and beyond what the blocks take in one
pass: thicknesses equal the oracle's rule and the task sizes its membership, exactly."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# tasks x 6 x steps entries: 288, 30000 (125 x 40), 36000 (125 x 48); 300000 particles exceed 1024 blocks of 256
@pytest.mark.parametrize("nt,steps,n", [((1, 1, 1), 48, 255), ((2, 1, 1), 48, 257), ((5, 5, 5), 40, 20000),
                                        ((5, 5, 5), 48, 20000), ((3, 2, 2), 64, 300000)])
@pytest.mark.parametrize("periodic", [True, False])
def test_thickness_and_sizes(vt, torch_cuda, oracle, nt, steps, n, periodic):
    p = np.random.default_rng(91).random((n, 3))
    thick, own, gh = vt.Context().vt_decompose(torch_cuda.from_numpy(p).cuda(), 0.0, 1.0, nt, border_factor=1.5,
                                               n_steps=steps, periodic=periodic)
    ref = oracle.autoborder(p, 0.0, 1.0, nt, border_factor=1.5, steps=steps, periodic=periodic)
    np.testing.assert_allclose(thick, ref, rtol=1e-14, atol=0)
    idx = oracle.task_index(p, 0.0, 1.0, nt)
    n_tasks = nt[0] * nt[1] * nt[2]
    assert np.array_equal(own, np.bincount((idx[:, 0] * nt[1] + idx[:, 1]) * nt[2] + idx[:, 2], minlength=n_tasks))
    for b in (0, n_tasks - 1):
        assert gh[b] == len(oracle.task_members(p, 0.0, 1.0, nt, thick, b, periodic=periodic)[1])
