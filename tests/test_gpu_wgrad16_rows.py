"""Filter gradient of 16-bit 3x3 layers by rows: strips of 8 columns, runs of rows, the deltas' and the map's rows beginning between dwords independently,
the ends of a caller's buffer, a strip's columns beside the rectangle - against sums in 64 bits."""
import numpy as np
import pytest
import torch

from ftp_synth.configs import conv, pool

pytestmark = pytest.mark.gpu


def _session(layers, batch, h, w, grid, groups, x, ws, dy):
    from paper_2409_09083_amd.harness import Session
    s = Session(layers, batch, layers[0].cin, h, w, grid, groups, "bf16")
    s.x.copy_(x)
    s.weights = ws
    s.dy.copy_(dy)
    s.step()
    torch.cuda.synchronize()
    return s


def _sums(dz, x):
    """sum over pixels of dz[co] * x[ci] moved by each tap, in 64 bits: the gradient, and the same of the magnitudes."""
    n, co, h, w = dz.shape
    xp = torch.nn.functional.pad(x, (1, 1, 1, 1))
    out = torch.empty(2, co, x.shape[1], 3, 3, dtype=torch.float64)
    a = dz.permute(1, 0, 2, 3).reshape(co, -1)
    for ky in range(3):
        for kx in range(3):
            b = xp[:, :, ky:ky + h, kx:kx + w].permute(1, 0, 2, 3).reshape(x.shape[1], -1)
            out[0, :, :, ky, kx] = a @ b.T
            out[1, :, :, ky, kx] = a.abs() @ b.abs().T
    return out


# (products of two bfloats are exact in fp32; each of as many additions as pixels rounds, or cuts, by at most 2^-23 of what is there)
@pytest.mark.parametrize("cin,cout,batch,h,w,grid", [
    (32, 32, 1, 3, 6, (1, 1)),            # one strip, fewer rows than a run has
    (64, 64, 1, 104, 104, (1, 1)),        # many shares, few strips: runs of rows
    (64, 64, 2, 30, 20, (1, 1)),          # an odd number of strips: halves in two images
    (32, 64, 3, 18, 76, (2, 8)),          # odd beginnings, two wavefronts to a strip pair
    (128, 96, 2, 26, 44, (3, 4)),         # ragged blocks of channels
    (96, 128, 5, 9, 38, (1, 8)),          # rows of 4 and 5
    (48, 40, 2, 21, 130, (2, 1)),         # the widest rows
    (256, 64, 4, 76, 76, (8, 8)),         # full launch, two strips a row
    (64, 128, 32, 60, 60, (3, 3)),        # full launch, three strips a row: the other kernel
])
@pytest.mark.parametrize("inner", [False, True])
def test_gradient_of_one_layer(cin, cout, batch, h, w, grid, inner):
    g = torch.Generator().manual_seed(cin + w)
    x = torch.randn(batch, cin, h, w, generator=g).bfloat16()
    dy = torch.randn(batch, cout, h, w, generator=g).bfloat16()
    wt = (torch.randn(cout, cin, 3, 3, generator=g) / (3 * cin ** 0.5)).bfloat16()
    layers, ws, at = (conv(cin, cout, 3, slope=1.0),), [wt.cuda()], 0
    if inner:                             # the same layer behind one that hands the map on: X in a stack's slot of the workspace
        one = torch.zeros(cin, cin, 1, 1)
        one[range(cin), range(cin)] = 1.0
        layers, ws, at = (conv(cin, cin, 1, slope=1.0),) + layers, [one.bfloat16().cuda()] + ws, cin * cin
    s = _session(layers, batch, h, w, grid, (len(layers),), x, ws, dy)
    got = s.wgrad.double().cpu()[at:].reshape(cout, cin, 3, 3)
    s.close()
    want = _sums(dy.double(), x.double())
    assert bool(((got - want[0]).abs() <= want[1] * (batch * h * w) * 2.0 ** -23).all())


@pytest.mark.parametrize("cin,cout,batch,h,w,grid", [
    (64, 64, 1, 60, 64, (1, 1)), (32, 64, 2, 24, 76, (2, 8)), (96, 32, 3, 20, 36, (5, 3)), (64, 64, 2, 8, 12, (2, 3)), (128, 64, 4, 40, 40, (8, 8)),
])
def test_gradient_through_a_pool(cin, cout, batch, h, w, grid):
    g = torch.Generator().manual_seed(cin + w)
    x = torch.randn(batch, cin, h, w, generator=g).bfloat16()
    dy = torch.randn(batch, cout, h // 2, w // 2, generator=g).bfloat16()
    wt = (torch.randn(cout, cin, 3, 3, generator=g) / (3 * cin ** 0.5)).bfloat16()
    s = _session((conv(cin, cout, 3, slope=1.0), pool(cout)), batch, h, w, grid, (2,), x, [wt.cuda()], dy)
    got = s.wgrad.double().cpu().reshape(cout, cin, 3, 3)
    # (the forward pass's own choice of the winners: its pooled values say which candidate they are)
    y = s.y.double().cpu()
    s.close()
    z = torch.nn.functional.conv2d(x.double(), wt.double(), padding=1)
    cand = z.reshape(batch, cout, h // 2, 2, w // 2, 2).permute(0, 1, 2, 4, 3, 5).reshape(batch, cout, h // 2, w // 2, 4)
    best = (cand - y[..., None]).abs().argmin(-1)
    two = cand.topk(2, -1).values
    clear = (two[..., 0] - two[..., 1]) > 0.02 * two[..., 0].abs() + 1e-2          # elsewhere the two candidates may round to one value
    dz = torch.zeros_like(cand).scatter_(-1, best[..., None], dy.double()[..., None])
    dz = dz.reshape(batch, cout, h // 2, w // 2, 2, 2).permute(0, 1, 2, 4, 3, 5).reshape(batch, cout, h, w)
    want = _sums(dz, x.double())
    # a window that is not clear may have another winner: its delta times the difference of two pixels, at most twice the largest |x|
    unclear = torch.where(clear, 0.0, dy.double().abs()).sum((0, 2, 3)) * 2 * x.double().abs().max()
    assert bool(((got - want[0]).abs() <= want[1] * (batch * h * w) * 2.0 ** -23 + unclear[:, None, None, None]).all())
    assert float(unclear.median() / want[0].abs().max()) < 5.0                     # ... and most of the sum is checked


def test_what_lies_beside_a_stack_stays_out_of_its_gradient():
    """One column of the map is not finite: only the gradients of the stacks that read it are not."""
    cin = cout = 32
    batch, h, w = 2, 8, 38
    g = torch.Generator().manual_seed(1)
    x = torch.randn(batch, cin, h, w, generator=g).bfloat16()
    x[:, :, :, 21] = float("inf")         # (grid of 1 x 2: the second stack's third column; the first one reads up to column 19)
    dy = torch.randn(batch, cout, h, w, generator=g).bfloat16()
    wt = torch.randn(cout, cin, 3, 3, generator=g).bfloat16()
    s = _session((conv(cin, cout, 3, slope=1.0),), batch, h, w, (1, 2), (1,), x, [wt.cuda()], dy)
    parts = s.partials.reshape(2, -1).cpu().numpy()
    s.close()
    assert np.isfinite(parts[0]).all() and not np.isfinite(parts[1]).any()
