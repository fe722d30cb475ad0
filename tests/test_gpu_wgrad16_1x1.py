"""Filter gradient of 16-bit 1x1 layers: the operands come from the maps in units of 8 pixels, so rows that begin between dwords (in X, in dZ, in
both), rows of a unit and of many, the ends of a caller's buffer, ragged channel blocks, both block widths and empty shares are where it can go wrong."""
import numpy as np
import pytest
import torch

from ftp_synth.configs import conv

pytestmark = pytest.mark.gpu


def _step(layers, batch, h, w, grid, groups, x, ws, dy):
    from paper_2409_09083_amd.harness import Session
    s = Session(layers, batch, layers[0].cin, h, w, grid, groups, "bf16")
    s.x.copy_(x)
    s.weights = ws
    s.dy.copy_(dy)
    s.step()
    torch.cuda.synchronize()
    got = s.wgrad.double().cpu()
    s.close()
    return got


@pytest.mark.parametrize("cin,cout,batch,h,w,grid", [
    (40, 32, 1, 6, 5, (1, 1)),            # rows of one unit, fewer steps than wavefronts
    (36, 40, 3, 8, 38, (1, 8)),           # 4 and 5 columns, odd beginnings
    (64, 64, 2, 7, 24, (1, 1)),           # whole units only
    (96, 72, 2, 13, 26, (2, 3)),          # ragged blocks, rows of 8 and 9
    (130, 68, 5, 20, 76, (4, 8)),         # the wide block's remainder
    (256, 128, 4, 76, 76, (8, 8)),        # the wide block: many stacks
    (128, 512, 8, 64, 64, (8, 8)),        # ... several of them a stack
    (48, 36, 1, 4, 126, (1, 1)),          # the widest rows
    (40, 36, 2, 6, 130, (1, 1)),          # wider ones: the other kernel
    (40, 32, 2, 5, 7, (1, 1)),            # odd channel stride: the other kernel
    (16, 64, 4, 66, 70, (2, 2)),          # few input channels: half a block
    (8, 32, 8, 64, 64, (3, 1)),
])
def test_gradient_of_one_layer(cin, cout, batch, h, w, grid):
    g = torch.Generator().manual_seed(5 + cin)
    x = torch.randn(batch, cin, h, w, generator=g).bfloat16()
    dy = torch.randn(batch, cout, h, w, generator=g).bfloat16()
    wt = (torch.randn(cout, cin, 1, 1, generator=g) / cin ** 0.5).bfloat16()
    got = _step((conv(cin, cout, 1, slope=1.0),), batch, h, w, grid, (1,), x, [wt.cuda()], dy).reshape(cout, cin)
    a, b = dy.double().permute(1, 0, 2, 3).reshape(cout, -1), x.double().permute(1, 0, 2, 3).reshape(cin, -1)
    # products of two bfloats are exact in fp32; each of n additions rounds (or cuts) by at most 2^-23 of what is there
    bound = (a.abs() @ b.abs().T) * a.shape[1] * 2.0 ** -23
    assert bool(((got - a @ b.T).abs() <= bound).all())


@pytest.mark.parametrize("h,w,grid", [(10, 38, (2, 4)), (9, 22, (1, 3)), (16, 50, (3, 3))])
def test_deltas_and_maps_of_other_parity(h, w, grid):
    """The delta of a layer inside a group lies in a stack's slot, X in the whole map: their rows begin between dwords independently."""
    cin, mid, cout, batch = 40, 40, 40, 3
    g = torch.Generator().manual_seed(h)
    x = torch.randn(batch, cin, h, w, generator=g).bfloat16()
    dy = torch.randn(batch, cout, h, w, generator=g).bfloat16()
    w0 = (torch.randn(mid, cin, 1, 1, generator=g) / cin ** 0.5).bfloat16()
    # an impulse filter hands the deltas on as they are: dW of the first layer is again a sum of exact products
    w1 = torch.zeros(cout, mid, 3, 3)
    w1[range(cout), range(mid), 1, 1] = 1.0
    layers = (conv(cin, mid, 1, slope=1.0), conv(mid, cout, 3, slope=1.0))
    got = _step(layers, batch, h, w, grid, (2,), x, [w0.cuda(), w1.bfloat16().cuda()], dy)[:mid * cin].reshape(mid, cin)
    a, b = dy.double().permute(1, 0, 2, 3).reshape(cout, -1), x.double().permute(1, 0, 2, 3).reshape(cin, -1)
    bound = (a.abs() @ b.abs().T) * a.shape[1] * 2.0 ** -23
    assert bool(((got - a @ b.T).abs() <= bound).all())


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_what_lies_beside_a_stack_stays_out_of_its_gradient(value):
    """One column of the map is not finite: only the gradients of the stacks that own it are not."""
    cin = cout = 40
    batch, h, w = 2, 8, 38
    g = torch.Generator().manual_seed(1)
    x = torch.randn(batch, cin, h, w, generator=g).bfloat16()
    x[:, :, :, 19] = value                # (grid of 1 x 2: the second stack's first column)
    dy = torch.randn(batch, cout, h, w, generator=g).bfloat16()
    wt = torch.randn(cout, cin, 1, 1, generator=g).bfloat16()
    from paper_2409_09083_amd.harness import Session
    s = Session((conv(cin, cout, 1, slope=1.0),), batch, cin, h, w, (1, 2), (1,), "bf16")
    s.x.copy_(x)
    s.weights = [wt.cuda()]
    s.dy.copy_(dy)
    s.step()
    torch.cuda.synchronize()
    parts = s.partials.reshape(2, -1).cpu().numpy()
    s.close()
    assert np.isfinite(parts[0]).all() and not np.isfinite(parts[1]).any()
