"""A training step whose deltas have become NaN or infinite, as in a run that diverges, takes about as long as any other: sums that
are not finite are computed again by whole workgroups, not by single lanes."""
import pytest
import torch

from ftp_synth.configs import conv, pool

pytestmark = pytest.mark.gpu

# layers, input size, batch, grid, storage type: one per kernel that computes such sums again
_NETS = {
    "delta": ((conv(64, 128, 1, slope=1.0),), 76, 8, (3, 3), "f32"),
    "gradient": ((conv(64, 128, slope=1.0),), 76, 8, (3, 3), "f32"),
    "gradient_pooled": ((conv(32, 64, slope=1.0), pool(64)), 152, 4, (4, 4), "f32"),
    "gradient_narrow": ((conv(16, 32, slope=1.0), conv(32, 32, slope=1.0)), 152, 4, (1, 1), "f32"),
    "first_layer_16": ((conv(3, 32, slope=1.0), pool(32)), 304, 4, (4, 4), "bf16"),
    "stem": ((conv(3, 64, 7, slope=1.0, stride=2),), 303, 4, (3, 3), "f32"),
    "delta5": ((conv(32, 64, 5, slope=1.0),), 76, 4, (3, 3), "f32"),
}


def _milliseconds(s):
    times = []
    for _ in range(6):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        s.step()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b))
    return min(times)


@pytest.mark.parametrize("net", sorted(_NETS))
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("everywhere", [True, False])
def test_time_of_a_step(net, value, everywhere):
    from paper_2409_09083_amd.harness import Session
    layers, hw, batch, grid, dtype = _NETS[net]
    s = Session(layers, batch, layers[0].cin, hw, hw, grid, (len(layers),), dtype=dtype)
    g = torch.Generator(device="cuda").manual_seed(1)
    s.x.uniform_(0, 1, generator=g)
    s.weights = [torch.randn((ly.cout, ly.cin, ly.k, ly.k), device="cuda", generator=g).to(s.x.dtype) / 20 if ly.kind == 0 else None for ly in layers]
    s.dy.normal_(generator=g)
    plain = _milliseconds(s)
    if everywhere:
        s.dy.fill_(value)
    else:
        s.dy.view(-1)[s.dy.numel() // 2 + 7] = value
    # (a workgroup multiplies twice at most, the second time at the rate of the fp32 instruction or of the vector units)
    assert _milliseconds(s) < 4.0 * plain + 0.05
    s.close()


@pytest.mark.parametrize("cin,cout", [(16, 32), (24, 40), (40, 72)])
@pytest.mark.parametrize("batch,h,w,grid,pooled", [(3, 9, 17, (1, 1), False), (5, 8, 8, (2, 2), False), (2, 20, 78, (1, 1), False), (9, 12, 10, (3, 2), False),
                                                   (2, 20, 78, (1, 1), True), (9, 12, 20, (3, 2), True)])
def test_filter_gradients(cin, cout, batch, h, w, grid, pooled):
    """fp32 3x3 filter gradients: infinities and NaN in both maps reach the entries they reach in a 64-bit sum, whatever lies beside
    them in a chunk; the other entries are as exact as ever."""
    from paper_2409_09083_amd.harness import Session
    layers = (conv(cin, cout, slope=1.0),) + ((pool(cout),) if pooled else ())
    s = Session(layers, batch, cin, h, w, grid, (len(layers),))
    g = torch.Generator().manual_seed(2)
    x = torch.rand(s.in_shape, generator=g) - 0.5
    wt = torch.randn((cout, cin, 3, 3), generator=g) / 12
    dy = torch.randn(s.out_shape, generator=g)
    hy, wy = dy.shape[2:]
    if not pooled:                                  # (a window's winner is not defined where its candidates are NaN)
        x[0, 3, h // 2, w - 3], x[batch - 1, 7, 3, 1], x[batch // 2, 9, h - 2, w // 2] = float("inf"), float("-inf"), float("nan")
    dy[0, 5, hy // 2, wy // 2], dy[batch - 1, 11, 1, wy - 2], dy[batch // 2, 17, hy - 2, 1] = float("inf"), float("nan"), float("-inf")
    s.x.copy_(x)
    s.dy.copy_(dy)
    s.weights = [wt.cuda()] + [None] * (len(layers) - 1)
    s.step()
    torch.cuda.synchronize()
    got = s.wgrad.cpu().reshape(wt.shape).double()
    s.close()
    # the same sums, one product per tap (zeros around the map are multiplied too)
    dz = dy.double()
    if pooled:
        y = torch.nn.functional.conv2d(x.double(), wt.double(), padding=1)
        _, idx = torch.nn.functional.max_pool2d(y, 2, return_indices=True)
        dz = torch.zeros(batch, cout, h * w, dtype=torch.float64).scatter_(2, idx.flatten(2), dz.flatten(2)).reshape(batch, cout, h, w)
    xp = torch.nn.functional.pad(x.double(), (1, 1, 1, 1))
    a = dz.transpose(0, 1).flatten(1)
    ref = torch.empty_like(got)
    mag = torch.empty_like(got)
    for t in range(9):
        v = xp[:, :, t // 3:t // 3 + h, t % 3:t % 3 + w].transpose(0, 1).flatten(1)
        ref[:, :, t // 3, t % 3] = (a[:, None, :] * v[None, :, :]).sum(-1)
        mag[:, :, t // 3, t % 3] = (a[:, None, :] * v[None, :, :]).abs().sum(-1)
    fin = torch.isfinite(ref)
    assert bool(fin.any()) and not bool(fin.all())
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    assert torch.equal(got[torch.isinf(ref)], ref[torch.isinf(ref)])
    # (one fp32 rounding, 2^-24 of the sum of magnitudes, per product summed)
    assert bool(((got - ref).abs()[fin] <= (batch * h * w + 8) * 2.0 ** -24 * mag[fin]).all())


@pytest.mark.parametrize("k", [3, 5, 7])
@pytest.mark.parametrize("batch", [2, 64])
def test_deltas_of_a_strided_stem(k, batch):
    """Tiles of 4 and of 16 rows of cells: the image's delta is not finite exactly where a tap reaches such a delta."""
    from tests.test_gpu_strided_stem import _run
    x, wt, dy, got = _run(conv(3, 20, k, slope=1.0, stride=2), batch, 69, 70, (1, 1), "f32", 9, poison=True)
    ref = torch.nn.grad.conv2d_input(x.shape, wt.double(), dy.double(), stride=2, padding=k // 2)
    mag = torch.nn.grad.conv2d_input(x.shape, wt.double().abs(), dy.double().abs().nan_to_num(0.0, 0.0, 0.0), stride=2, padding=k // 2)
    fin = torch.isfinite(ref)
    assert torch.equal(torch.isfinite(got), fin) and not bool(fin.all())
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    # (one fp32 rounding, 2^-24 of the sum of magnitudes, per product summed)
    assert bool(((got.double() - ref).abs()[fin] <= (k * k * 20 + 4) * 2.0 ** -24 * mag[fin] + 1e-30).all())
