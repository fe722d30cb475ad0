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


@pytest.mark.parametrize("cin,cout", [(1, 5), (2, 33), (3, 32)])
@pytest.mark.parametrize("batch,h,w,grid", [(2, 16, 32, (1, 1)), (3, 44, 100, (1, 1)), (4, 128, 192, (2, 1))])
def test_filter_gradient_against_64_bits(cin, cout, batch, h, w, grid):
    """The gradient is an fp32 sum of exact products: nothing of it is rounded to 16 bits."""
    import torch
    from paper_2409_09083_amd import binding as B
    from paper_2409_09083_amd.harness import Session
    g = torch.Generator().manual_seed(6)
    s = Session((conv(cin, cout, slope=1.0), pool(cout)), batch, cin, h, w, grid, (2,), dtype="bf16")
    x = torch.rand(s.in_shape, generator=g).bfloat16()
    wt = (torch.randn((cout, cin, 3, 3), generator=g) / 5).bfloat16()
    dy = torch.randn(s.out_shape, generator=g).bfloat16()
    s.load(x=x.float().numpy(), weights=[wt.float().numpy(), None], dy=dy.float().numpy())
    s.step()
    torch.cuda.synchronize()
    # (the winners as the forward pass decided them)
    win = (torch.from_numpy(s.get_boundary(2, B.FTP_BUF_MASK)).long() >> 1) & 3
    dz = torch.zeros((batch, cout, h, w), dtype=torch.float64)
    for q in range(4):
        dz[:, :, q >> 1::2, q & 1::2] = torch.where(win == q, dy.double(), 0.0)
    ref = torch.nn.grad.conv2d_weight(x.double(), wt.shape, dz, padding=1)
    err = float((s.wgrad.cpu().double().reshape(ref.shape) - ref).norm() / ref.norm())
    # (one rounding of 2^-24 per 16 pixels summed at most, all of one sign; random ones leave 1e-7 or so)
    assert err < 1e-6, err
    s.close()
