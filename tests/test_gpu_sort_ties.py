"""The sort's routes with equal keys (pairs of particles closer than the keys' quantum, 2^-16 of the
box, anywhere in the input, so within and across the compared route's chunks of 64 and the radix
tiles), and with long runs of equal digits (half of the particles in a smooth-edged clump) on the
routes of a million.  A particle lost, doubled or out of place shows in the volumes: they fill the box,
and a sample's are the oracle's.  Tolerance: pairs a quantum apart give neighbours planes at angles of
1e-4 to 1e-3 of a right one, whose vertices round by the inverse of it, squared at worst: 1e-16 of
1e8, 1e-8 of a volume."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _check(vt, torch_cuda, oracle, p, own, rows):
    items = vt.whole_box(own, 0.0, 1.0, periodic=False, walls=63)
    items[0]["n_ghost"] = len(p) - own
    ctx = vt.Context().vt_build(torch_cuda.from_numpy(p).cuda(), items)
    assert ctx.vt_query()[0] == 0
    vol = ctx.vt_cells().volume.cpu().numpy()
    if own == len(p):
        assert abs(vol.sum() - 1.0) <= 1e-8
    ref = oracle.local_cells(p, 0.0, 1.0, rows, periodic=False)
    np.testing.assert_allclose(vol[rows], ref.volume, rtol=1e-8, atol=0)


@pytest.mark.parametrize("ghosts", [0, 1])
@pytest.mark.parametrize("n", [64, 130, 4096, 4097, 20480, 20481, 40000])
def test_equal_keys(vt, torch_cuda, oracle, n, ghosts):
    rng = np.random.default_rng(n)
    half = (3 * n) // 8
    p = rng.random((n - half, 3))
    twin = p[:half] + 2.0 ** -18 * rng.uniform(-1.0, 1.0, (half, 3))
    p = np.clip(np.concatenate([p, twin]), 1e-9, 1.0 - 1e-9)[rng.permutation(n)]
    own = n - n // 3 if ghosts else n
    q = np.floor(p * 65536.0).astype(np.int64)
    assert len(np.unique(q, axis=0)) < n - n // 8
    _check(vt, torch_cuda, oracle, p, own, rng.permutation(own)[:200])


@pytest.mark.parametrize("ghosts", [0, 1])
@pytest.mark.parametrize("n", [300000, 1048576, 1048577])
def test_clump(vt, torch_cuda, oracle, n, ghosts):
    rng = np.random.default_rng(n)
    p = rng.random((n, 3))
    p[::2] = np.clip(0.4 + 0.05 * rng.standard_normal((len(p[::2]), 3)), 0.01, 0.99)
    own = n - n // 3 if ghosts else n
    _check(vt, torch_cuda, oracle, p, own, rng.permutation(own)[:200])
