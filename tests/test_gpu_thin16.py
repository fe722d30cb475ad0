"""Gradients of 16-bit 3x3 first layers with a fused pool against the oracle: column blocks of 1 to 3
steps, last rows and columns that fill a chunk partly, odd strides between channels, channel counts around a block of 32."""
import pytest

from ftp_synth.configs import Config, conv, pool
from tests import parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin,cout", [(1, 5), (2, 33), (3, 32), (4, 40)])
@pytest.mark.parametrize("batch,h,w,grid", [(2, 16, 32, (1, 1)), (3, 44, 100, (1, 1)), (2, 54, 226, (1, 1)), (2, 60, 142, (2, 3))])
def test_gradients(oracle, cin, cout, batch, h, w, grid):
    P.check_case(oracle, Config("thin16", batch, cin, h, w, (conv(cin, cout), pool(cout)), grid, (2,), "bf16"))


def test_non_finite_deltas_reach_only_the_pixels_with_a_tap():
    """Infinite and NaN deltas through the pool: the image's delta is non-finite exactly where the reference's is."""
    import torch
    from paper_2409_09083_amd.harness import Session
    g = torch.Generator().manual_seed(4)
    s = Session((conv(3, 24), pool(24)), 2, 3, 48, 60, (1, 2), (2,), dtype="bf16")
    x = torch.randn(s.in_shape, generator=g).bfloat16()
    w = (torch.randn((24, 3, 3, 3), generator=g) / 5).bfloat16()
    dy = torch.randn(s.out_shape, generator=g).bfloat16()
    dy[0, 3, 4, 5], dy[0, 9, 20, 14], dy[1, 0, 0, 0], dy[1, 7, -1, -1] = float("inf"), float("-inf"), float("nan"), float("inf")
    s.load(x=x.float().numpy(), weights=[w.float().numpy(), None], dy=dy.float().numpy())
    s.step()
    torch.cuda.synchronize()
    got = torch.from_numpy(s.to_np(s.dx).astype("float32")).reshape(x.shape)
    xr = x.float().requires_grad_(True)
    y = torch.nn.functional.max_pool2d(torch.nn.functional.leaky_relu(torch.nn.functional.conv2d(xr, w.float(), padding=1), 0.1).bfloat16().float(), 2)
    (ref,) = torch.autograd.grad(y, xr, dy.float())
    fin = torch.isfinite(ref)
    assert torch.equal(torch.isfinite(got), fin) and not bool(fin.all())
    # (a 16-bit map's rounding, twice)
    assert float(((got - ref).abs() / (ref.abs() + 1))[fin].max()) < 2.0 ** -7
    s.close()
