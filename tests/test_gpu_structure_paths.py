"""The structure's two routes (cells written from their records, cells rebuilt) against each other's
neighbours: bounded worlds mix both in one batch (interior cells have only particle faces, border
cells walls), an area threshold that drops faces sends cells to the rebuild, counts around the
batches of 16 and of a block, ids of every sign.  Faces and loops are whole numbers and must agree
exactly with the oracle's; vertices within 1e-12 of the box (three well-conditioned planes)."""
import numpy as np
import pytest

from test_gpu_structure import _against_oracle, _host, _whole_cell_checks

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 130, 1025])
def test_bounded_world_mixes_routes(vt, torch_cuda, oracle, n):
    p = np.random.default_rng(81).random((n, 3))
    ctx = vt.Context().vt_build(torch_cuda.from_numpy(p).cuda(), vt.whole_box(n, 0.0, 1.0, periodic=False, walls=63),
                                want_faces=True)
    h = _host(ctx.vt_structure())
    assert ctx.vt_query()[0] == 0
    _against_oracle(oracle, h, range(min(n, 60)), p, 0.0, 1.0, periodic=False)


@pytest.mark.parametrize("eps", [1e-12, 1e-3])
def test_dropped_faces(vt, torch_cuda, eps):
    p = np.random.default_rng(82).random((3000, 3))
    ctx = vt.Context().vt_build(torch_cuda.from_numpy(p).cuda(), vt.whole_box(3000, 0.0, 1.0), want_faces=True,
                                area_eps=eps)
    cells = ctx.vt_cells()
    h = _host(ctx.vt_structure())
    assert ctx.vt_query()[0] == 0
    ids = h["face_nbr"]
    assert np.array_equal(ids, cells.nbr_ids.cpu().numpy())
    assert np.array_equal(h["face_off"], cells.nbr_off.cpu().numpy())
    entries = np.diff(h["loop_off"])
    assert entries.min() >= 3
    closed = np.add.reduceat(entries, h["face_off"][:-1]) == 3 * np.diff(h["vert_off"])
    if eps > 1e-9:
        assert (~closed).any()
    else:
        _whole_cell_checks(h, p, cells)


def test_ids_of_every_sign(vt, torch_cuda):
    n = 2000
    p = np.random.default_rng(83).random((n, 3))
    gid = np.random.default_rng(84).permutation(n).astype(np.int32) - n // 2
    ctx = vt.Context().vt_build(torch_cuda.from_numpy(p).cuda(), vt.whole_box(n, 0.0, 1.0),
                                global_id=torch_cuda.from_numpy(gid).cuda(), want_faces=True)
    h = _host(ctx.vt_structure())
    assert ctx.vt_query()[0] == 0
    key = (h["face_nbr"].astype(np.int64) + 16) & 0xFFFFFFFF
    first = np.zeros(len(key), bool)
    first[h["face_off"][:-1]] = True
    assert np.all((np.diff(key) > 0) | first[1:])
