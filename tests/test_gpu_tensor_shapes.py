"""Grid tensors on every remainder of the radix-8 passes, with lines too few or too short for a
block, with a field that shares memory with the output, and with an output aligned to 8 bytes only.

Tolerance: a transform of n points in FP64 is within a few eps log2(n) of the exact one, relative to
the spectrum's 2-norm (eps = 1.1e-16, log2 n <= 21 here: 1e-14 with a factor of five), and the
largest component is at least 1 / sqrt(n) = 1/1449 of that norm for the fields drawn: 1.5e-11."""
import numpy as np
import pytest

from paper_1601_06429_amd import workloads as wl

pytestmark = pytest.mark.gpu
RTOL = 1.5e-11


def _ctx(vt, torch_cuda):
    w = wl.uniform4096()
    return w, vt.Context().vt_build(torch_cuda.from_numpy(w.pos).cuda(), vt.whole_box(w.n, w.box_lo, w.box_hi))


@pytest.mark.parametrize("kind", ["tidal", "hessian"])
@pytest.mark.parametrize("shape", [(2, 4, 2), (4, 2, 8), (8, 16, 2), (16, 32, 4), (64, 8, 16), (128, 256, 8),
                                   (32, 2, 1024), (512, 64, 8), (2, 2048, 2), (1024, 8, 2), (16, 4096, 2), (64, 256, 128), (1024, 1024, 2)])
def test_every_line_length(vt, torch_cuda, oracle, kind, shape):
    w, ctx = _ctx(vt, torch_cuda)
    f = 2.0 + np.random.default_rng(57).random(shape)
    k = vt.TENSOR_TIDAL if kind == "tidal" else vt.TENSOR_HESSIAN
    ref = oracle.grid_tensor(f, w.box_hi - w.box_lo, kind)
    out = ctx.vt_grid_tensor(torch_cuda.from_numpy(f).cuda(), k).cpu().numpy()
    assert np.max(np.abs(out - ref)) <= RTOL * max(np.abs(ref).max(), 1e-300)


@pytest.mark.parametrize("at", [0, 1, 2, 3, 4, 5, "between"])
def test_field_inside_the_output(vt, torch_cuda, oracle, at):
    w, ctx = _ctx(vt, torch_cuda)
    shape, n = (16, 8, 32), 16 * 8 * 32
    f = 2.0 + np.random.default_rng(58).random(shape)
    out = torch_cuda.zeros(6 * n, dtype=torch_cuda.float64, device="cuda")
    first = 2 * n - n // 2 + 1 if at == "between" else at * n
    field = out[first:first + n].view(shape)
    field.copy_(torch_cuda.from_numpy(f))
    got = ctx.vt_grid_tensor(field, vt.TENSOR_TIDAL, out=out.view((6,) + shape)).cpu().numpy()
    ref = oracle.grid_tensor(f, w.box_hi - w.box_lo, "tidal")
    assert np.max(np.abs(got - ref)) <= RTOL * np.abs(ref).max()


def test_output_aligned_to_eight_bytes(vt, torch_cuda, oracle):
    w, ctx = _ctx(vt, torch_cuda)
    shape, n = (8, 16, 32), 8 * 16 * 32
    f = 2.0 + np.random.default_rng(59).random(shape)
    buf = torch_cuda.zeros(7 * n + 4, dtype=torch_cuda.float64, device="cuda")
    field, out = buf[6 * n + 3:7 * n + 3].view(shape), buf[1:6 * n + 1].view((6,) + shape)
    field.copy_(torch_cuda.from_numpy(f))
    got = ctx.vt_grid_tensor(field, vt.TENSOR_HESSIAN, out=out).cpu().numpy()
    ref = oracle.grid_tensor(f, w.box_hi - w.box_lo, "hessian")
    assert np.max(np.abs(got - ref)) <= RTOL * np.abs(ref).max()
    assert float(buf[0]) == 0.0 and float(buf[6 * n + 1]) == 0.0
