"""Delta at the image side of a strided stem (at most 4 input channels) on the matrix cores: single layers against 64-bit sums, few
and many workgroups (tiles of 4 and of 16 rows of cells), odd maps, channel counts around a stage; infinities and NaN."""
import numpy as np
import pytest
import torch

from ftp_synth.configs import conv

pytestmark = pytest.mark.gpu


def _run(ly, batch, h, w, grid, dtype, seed, poison=False):
    from paper_2409_09083_amd.harness import Session
    g = torch.Generator().manual_seed(seed)
    s = Session((ly,), batch, ly.cin, h, w, grid, (1,), dtype=dtype)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = (torch.rand(s.in_shape, generator=g) - 0.5).to(td)
    wt = (torch.randn((ly.cout, ly.cin, ly.k, ly.k), generator=g) / np.sqrt(ly.cin * ly.k * ly.k)).to(td)
    dy = torch.randn(s.out_shape, generator=g).to(td)
    if poison:
        dy[0, 1, 2, 3], dy[0, 4, 7, 1], dy[-1, 0, -1, -1] = float("inf"), float("-inf"), float("nan")
    s.load(x=x.float().numpy(), weights=[wt.float().numpy()], dy=dy.float().numpy())
    s.step()
    torch.cuda.synchronize()
    got = torch.from_numpy(np.asarray(s.to_np(s.dx), dtype=np.float32).reshape(x.shape))
    s.close()
    return x, wt, dy, got


@pytest.mark.parametrize("k", [3, 5, 7])
@pytest.mark.parametrize("cin,cout", [(1, 3), (2, 8), (3, 17), (4, 24)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_delta(k, cin, cout, dtype):
    ly = conv(cin, cout, k, slope=1.0, stride=2)
    for i, (batch, h, w, grid) in enumerate([(1, 9, 7, (1, 1)), (2, 45, 71, (2, 3)), (64, 69, 70, (1, 1))]):
        x, wt, dy, got = _run(ly, batch, h, w, grid, dtype, 3 + i)
        op = lambda a, b: torch.nn.grad.conv2d_input(x.shape, b.double(), a.double(), stride=2, padding=k // 2)
        ref = op(dy, wt)
        # one fp32 rounding (2^-24 of the sum of magnitudes) per product summed, and the rounding of a 16-bit map (2^-9, kept at 2^-8)
        bound = (k * k * cout + 4) * 2.0 ** -24 * op(dy.abs(), wt.abs()) + (2.0 ** -8 * ref.abs() if dtype == "bf16" else 0.0) + 1e-30
        err = (got.double() - ref).abs()
        assert bool((err <= bound).all()), (batch, float((err / bound).max()))


@pytest.mark.parametrize("k", [3, 7])
def test_non_finite_deltas_reach_only_the_pixels_with_a_tap(k):
    x, wt, dy, got = _run(conv(3, 12, k, slope=1.0, stride=2), 2, 40, 52, (2, 2), "f32", 9, poison=True)
    ref = torch.nn.grad.conv2d_input(x.shape, wt.double(), dy.double(), stride=2, padding=k // 2)
    # (the reference multiplies what lies outside the taps by nothing; where it is finite, ours is)
    assert torch.equal(torch.isfinite(got), torch.isfinite(ref))
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    fin = torch.isfinite(ref)
    assert float(((got.double() - ref).abs() / (ref.abs() + 1))[fin].max()) < 1e-5
