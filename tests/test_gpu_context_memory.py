"""What a context holds after builds of different sizes, with and without facets: the facet arrays are
there for the cells of the builds that ask for them only, whichever came first.  Held memory is the
device's free memory before less after; a build of the larger size alone is the yardstick, and 64 MiB
is a tenth of what its facet arrays would take (twice what the smaller build's part comes to)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

BIG, SMALL = 500000, 1000


@pytest.mark.parametrize("first", [(SMALL, True), (BIG, False)])
def test_facet_arrays(vt, torch_cuda, first):
    pos = {n: torch_cuda.from_numpy(np.random.default_rng(n).random((n, 3))).cuda() for n in (BIG, SMALL)}

    def held(*builds):
        torch_cuda.cuda.synchronize()
        before = torch_cuda.cuda.mem_get_info()[0]
        ctx = vt.Context()
        for n, faces in builds:
            ctx.vt_build(pos[n], vt.whole_box(n, 0.0, 1.0), want_faces=faces)
            assert ctx.vt_query()[0] == 0
        return before - torch_cuda.cuda.mem_get_info()[0]

    held((SMALL, False))   # what the runtime keeps for itself
    alone = held((BIG, False))
    second = (BIG, False) if first == (SMALL, True) else (SMALL, True)
    assert held(first, second) <= alone + (64 << 20)
