"""fp32 3x3 filter gradient on the bfloat matrix cores: against 64-bit sums at the edges of its chunks (rectangles of one
group of pixels, one more, several column blocks, several images to a chunk) and blocks; infinities and NaN."""
import pytest
import torch

from ftp_synth.configs import conv, pool
from tests.test_gpu_delta_split import _load, _session

pytestmark = pytest.mark.gpu


def _grad(x, ws, dy, pooled, dtype, slope=1.0):
    w = ws[0].to(dtype).requires_grad_(True)
    y = torch.nn.functional.leaky_relu(torch.nn.functional.conv2d(x.to(dtype), w, padding=1), slope)
    if pooled:
        y = torch.nn.functional.max_pool2d(y, 2)
    (g,) = torch.autograd.grad(y, w, dy.to(dtype))
    return g


@pytest.mark.parametrize("cin,cout", [(16, 32), (33, 36), (24, 70), (72, 132)])
@pytest.mark.parametrize("batch,h,w,grid,pooled", [(3, 9, 17, (1, 1), False)] + [s + (p,) for p in (False, True) for s in (
    (5, 8, 8, (2, 2)), (2, 20, 78, (1, 1)), (4, 26, 26, (2, 1)), (9, 12, 10, (3, 2)))])
def test_against_64_bits(cin, cout, batch, h, w, grid, pooled):
    layers = (conv(cin, cout, slope=1.0),) + ((pool(cout),) if pooled else ())
    s, x, ws, dy = _session(layers, batch, h, w, grid, 3)
    _load(s, x, ws, dy)
    s.step()
    torch.cuda.synchronize()
    ref = _grad(x, ws, dy, pooled, torch.float64)
    # every sum has batch * h * w terms; a term is rounded into a partial sum once per 8 terms and product of planes
    dz = torch.nn.functional.interpolate(dy.abs(), scale_factor=2) if pooled else dy.abs()
    mag = torch.nn.grad.conv2d_weight(x.abs().double(), ws[0].shape, dz.double(), padding=1)
    bound = (6 * (batch * h * w // 8 + 8) + 1) * 2.0 ** -24 * mag
    err = (s.wgrad.cpu().double().reshape(ref.shape) - ref).abs()
    assert bool((err <= bound).all())
    # (without one of the three smallest products random sums are off by 2.4e-6)
    assert float(err.norm() / ref.norm()) < 1e-6
    s.close()


@pytest.mark.parametrize("pooled", [False, True])
def test_non_finite_values_come_out_as_fp32_sums_give_them(pooled):
    layers = (conv(24, 40),) + ((pool(40),) if pooled else ())
    s, x, ws, dy = _session(layers, 2, 20, 28, (1, 1), 5)
    dy[0, 3, 4, 5] = float("inf")
    dy[1, 9, 5, 7] = float("nan")
    dy[1, 30, 5, 9] = 3.4e38                        # above the largest bfloat
    _load(s, x, ws, dy)
    s.step()
    torch.cuda.synchronize()
    ref = _grad(x, ws, dy, pooled, torch.float32, 0.1)
    got = s.wgrad.cpu().reshape(ref.shape)
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    assert torch.equal(got[torch.isinf(ref)], ref[torch.isinf(ref)])
    fin = torch.isfinite(ref)
    assert torch.equal(torch.isfinite(got), fin)
    assert float(((got - ref).abs() / (ref.abs() + 1))[fin].max()) < 1e-4
    s.close()
