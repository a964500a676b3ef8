"""The sort's three routes (all pairs compared up to 20480 particles, radix passes with the tiles'
counts summed by the scatter up to 256 tiles of 4096, and scanned beyond) at their edges, with and
without buffer particles, uniform or with half of the particles in a small clump (long runs of equal
digits).  Keys are distinct, so the sorted order, and with it every cell, does not depend on the
input's order: a shuffled input gives the same volumes bit for bit, and they fill the box.  (A clump's
sharp edge among a million particles gives cells beyond the face capacity: then both orders are
refused alike.)"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("clump", [True, False])
@pytest.mark.parametrize("ghosts", [0, 1])
@pytest.mark.parametrize("n", [9, 63, 64, 65, 255, 257, 1025, 4095, 4096, 4097, 8192, 20480, 20481, 1048576, 1048577])
def test_order_of_input_does_not_matter(vt, torch_cuda, n, ghosts, clump):
    rng = np.random.default_rng(n)
    p = rng.random((n, 3))
    if clump:
        p[::2] = 0.4 + 0.05 * p[::2]
    own = n - n // 3 if ghosts else n
    perm = np.concatenate([rng.permutation(own), own + rng.permutation(n - own)])
    items = vt.whole_box(own, 0.0, 1.0, periodic=False, walls=63)
    items[0]["n_ghost"] = n - own
    vols, codes = [], []
    for x in (p, p[perm]):
        ctx = vt.Context().vt_build(torch_cuda.from_numpy(x).cuda(), items)
        codes.append(ctx.vt_query()[0])
        if codes[-1] == 0:
            vols.append(ctx.vt_cells().volume.cpu().numpy())
    assert codes[0] == codes[1] and (codes[0] == 0 or (clump and n > 1000000 and codes[0] == 6))
    if codes[0] == 0:
        assert np.array_equal(vols[0][perm[:own]], vols[1])
        if not ghosts:
            assert abs(vols[0].sum() - 1.0) < 1e-12
