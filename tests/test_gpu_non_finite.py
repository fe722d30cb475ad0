"""A training step whose deltas have become NaN or infinite, as in a run that diverges, takes about as long as any other: sums that
are not finite are computed again by whole workgroups, not by single lanes."""
import pytest
import torch

from ftp_synth.configs import conv, pool

pytestmark = pytest.mark.gpu

# layers, input size, batch, grid, storage type: one per kernel that computes such sums again
_NETS = {
    "delta": ((conv(64, 128, 1, slope=1.0),), 76, 8, (3, 3), "f32"),
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
