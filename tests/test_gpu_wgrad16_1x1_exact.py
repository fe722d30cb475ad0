"""Filter gradient of 16-bit 1x1 layers: the operands come from the maps in units of 8 pixels, so rows that begin between dwords (in X, in dZ, in
both), rows of a unit and of many, the ends of a caller's buffer, ragged channel blocks, both block widths and empty shares are where it can go wrong.
Operands are small whole numbers: every sum is exact in fp32, in any order, and a pixel that is missed, doubled or moved shows."""
import pytest
import torch

from ftp_synth.configs import conv
from paper_2409_09083_amd import binding as B

pytestmark = pytest.mark.gpu


def _whole(shape, most, g):
    return torch.randint(-most, most + 1, shape, generator=g).bfloat16()


def _gradients(layers, batch, h, w, grid, groups, x, ws, dy):
    """Joined with the delta where that applies, and in launches of their own (timing records on); the first layer's kernel there."""
    from paper_2409_09083_amd.harness import Session
    out = []
    for records in (False, True):
        s = Session(layers, batch, layers[0].cin, h, w, grid, groups, "bf16")
        s.x.copy_(x)
        s.weights = ws
        s.dy.copy_(dy)
        if records:
            B.ftp_profile(s.plan, 1)
        s.step()
        torch.cuda.synchronize()
        out.append(s.wgrad.double().cpu())
        if records:
            kernel = [r["kernel"].split("<")[0] for r in B.ftp_profile_read(s.plan) if r["pass"] == "wgrad" and r["layer"] == 0]
        s.close()
    return out, kernel


@pytest.mark.parametrize("cin,cout,batch,h,w,grid,kernel", [
    (40, 32, 1, 6, 5, (1, 1), "k_wgrad16_1x1"),            # rows of one unit, fewer steps than wavefronts
    (36, 40, 3, 8, 38, (1, 8), "k_wgrad16_1x1"),           # 4 and 5 columns, odd beginnings
    (64, 64, 2, 7, 24, (1, 1), "k_wgrad16_1x1"),           # whole units only
    (96, 72, 2, 13, 26, (2, 3), "k_wgrad16_1x1"),          # ragged blocks, rows of 8 and 9
    (130, 68, 5, 20, 76, (4, 8), "k_wgrad16_1x1"),         # the wide block's remainder
    (256, 128, 4, 76, 76, (8, 8), "k_wgrad16_1x1"),        # the wide block: many stacks
    (128, 512, 8, 64, 64, (8, 8), "k_wgrad16_1x1"),        # ... several of them a stack
    (48, 36, 1, 4, 126, (1, 1), "k_wgrad16_1x1"),          # the widest rows
    (40, 36, 2, 6, 130, (1, 1), "k_wgrad_mfma"),           # wider ones: the other kernel
    (40, 32, 2, 5, 7, (1, 1), "k_wgrad_mfma"),             # odd channel stride: the other kernel
    (16, 64, 4, 66, 70, (2, 2), "k_wgrad16_1x1"),          # few input channels: half a block
    (8, 32, 10, 128, 126, (3, 1), "k_wgrad16_1x1"),
])
def test_gradient_of_one_layer(cin, cout, batch, h, w, grid, kernel):
    g = torch.Generator().manual_seed(5 + cin)
    x, dy = _whole((batch, cin, h, w), 4, g), _whole((batch, cout, h, w), 2, g)
    wt = (torch.randn(cout, cin, 1, 1, generator=g) / cin ** 0.5).bfloat16()
    got, taken = _gradients((conv(cin, cout, 1, slope=1.0),), batch, h, w, grid, (1,), x, [wt.cuda()], dy)
    a, b = dy.double().permute(1, 0, 2, 3).reshape(cout, -1), x.double().permute(1, 0, 2, 3).reshape(cin, -1)
    assert taken == [kernel] and 8 * a.shape[1] < 2 ** 24
    for v in got:
        assert torch.equal(v.reshape(cout, cin), a @ b.T)


@pytest.mark.parametrize("h,w,grid", [(10, 38, (2, 4)), (9, 22, (1, 3)), (16, 50, (3, 3))])
def test_deltas_and_maps_of_other_parity(h, w, grid):
    """The delta of a layer inside a group lies in a stack's slot, X in the whole map: their rows begin between dwords independently."""
    cin, mid, cout, batch = 40, 40, 40, 3
    g = torch.Generator().manual_seed(h)
    x, dy = _whole((batch, cin, h, w), 4, g), _whole((batch, cout, h, w), 2, g)
    w0 = (torch.randn(mid, cin, 1, 1, generator=g) / cin ** 0.5).bfloat16()
    # an impulse filter hands the deltas on as they are: dW of the first layer is again a sum of exact products
    w1 = torch.zeros(cout, mid, 3, 3)
    w1[range(cout), range(mid), 1, 1] = 1.0
    layers = (conv(cin, mid, 1, slope=1.0), conv(mid, cout, 3, slope=1.0))
    got, taken = _gradients(layers, batch, h, w, grid, (2,), x, [w0.cuda(), w1.bfloat16().cuda()], dy)
    a, b = dy.double().permute(1, 0, 2, 3).reshape(cout, -1), x.double().permute(1, 0, 2, 3).reshape(cin, -1)
    assert taken == ["k_wgrad16_1x1"]
    for v in got:
        assert torch.equal(v[:mid * cin].reshape(mid, cin), a @ b.T)
