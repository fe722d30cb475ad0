"""Filter gradient of 16-bit 3x3 layers by rows: strips of 8 columns, runs of rows, the deltas' and the map's rows beginning between dwords independently,
the ends of a caller's buffer, a strip's columns beside the rectangle.  Operands are small whole numbers: every sum is exact in fp32, in any order, and a
pixel that is missed, doubled or moved shows; in launches of their own (timing records on) and joined with the delta."""
import pytest
import torch

from ftp_synth.configs import conv, pool
from paper_2409_09083_amd import binding as B

pytestmark = pytest.mark.gpu


def _session(layers, batch, h, w, grid, groups, x, ws, dy, records=False):
    from paper_2409_09083_amd.harness import Session
    s = Session(layers, batch, layers[0].cin, h, w, grid, groups, "bf16")
    s.x.copy_(x)
    s.weights = ws
    s.dy.copy_(dy)
    if records:
        B.ftp_profile(s.plan, 1)
    s.step()
    torch.cuda.synchronize()
    return s


def _whole(shape, most, g):
    return torch.randint(-most, most + 1, shape, generator=g).bfloat16()


def _gradients(layers, batch, h, w, grid, x, ws, dy, at):
    """Of the layer whose filter begins at `at`: joined with the delta where that applies, and apart; the kernel that it takes apart."""
    out = []
    for records in (False, True):
        s = _session(layers, batch, h, w, grid, (len(layers),), x, ws, dy, records)
        out.append(s.wgrad.double().cpu()[at:])
        if records:
            kernel = [r["kernel"] for r in B.ftp_profile_read(s.plan) if r["pass"] == "wgrad" and r["kernel"].startswith("k_wgrad_mfma16<")]
        s.close()
    return out, kernel


def _sums(dz, x):
    """sum over pixels of dz[co] * x[ci] moved by each tap, in 64 bits."""
    n, co, h, w = dz.shape
    xp = torch.nn.functional.pad(x, (1, 1, 1, 1))
    out = torch.empty(co, x.shape[1], 3, 3, dtype=torch.float64)
    a = dz.permute(1, 0, 2, 3).reshape(co, -1)
    for ky in range(3):
        for kx in range(3):
            out[:, :, ky, kx] = a @ xp[:, :, ky:ky + h, kx:kx + w].permute(1, 0, 2, 3).reshape(x.shape[1], -1).T
    return out


@pytest.mark.parametrize("cin,cout,batch,h,w,grid,rows", [
    (32, 32, 1, 3, 6, (1, 1), True),            # one strip, fewer rows than a run has
    (64, 64, 1, 104, 104, (1, 1), True),        # many shares, few strips: runs of rows
    (64, 64, 2, 30, 20, (1, 1), True),          # an odd number of strips: halves in two images
    (32, 64, 3, 18, 76, (2, 8), True),          # odd beginnings, two wavefronts to a strip pair
    (128, 96, 2, 26, 44, (3, 4), True),         # ragged blocks of channels
    (96, 128, 5, 9, 38, (1, 8), True),          # rows of 4 and 5
    (48, 40, 2, 21, 130, (2, 1), True),         # the widest rows
    (256, 64, 4, 76, 76, (8, 8), True),         # full launch, two strips a row
    (64, 128, 32, 60, 60, (3, 3), False),       # full launch, three strips a row: the other kernel
])
@pytest.mark.parametrize("inner", [False, True])
def test_gradient_of_one_layer(cin, cout, batch, h, w, grid, rows, inner):
    g = torch.Generator().manual_seed(cin + w)
    x, dy = _whole((batch, cin, h, w), 4, g), _whole((batch, cout, h, w), 2, g)
    wt = (torch.randn(cout, cin, 3, 3, generator=g) / (3 * cin ** 0.5)).bfloat16()
    layers, ws, at = (conv(cin, cout, 3, slope=1.0),), [wt.cuda()], 0
    if inner:                             # the same layer behind one that hands the map on: X in a stack's slot of the workspace
        one = torch.zeros(cin, cin, 1, 1)
        one[range(cin), range(cin)] = 1.0
        layers, ws, at = (conv(cin, cin, 1, slope=1.0),) + layers, [one.bfloat16().cuda()] + ws, cin * cin
    got, kernel = _gradients(layers, batch, h, w, grid, x, ws, dy, at)
    want = _sums(dy.double(), x.double())
    assert 8 * batch * h * w < 2 ** 24 and kernel == ["k_wgrad_mfma16<%d, 0, %s, %s>" % (1 if cin <= 32 else 2, "true" if inner else "false", "true" if rows else "false")]
    for v in got:
        assert torch.equal(v.reshape(want.shape), want)


@pytest.mark.parametrize("cin,cout,batch,h,w,grid", [
    (64, 64, 1, 60, 64, (1, 1)), (32, 64, 2, 24, 76, (2, 8)), (96, 32, 3, 20, 36, (5, 3)), (64, 64, 2, 8, 12, (2, 3)), (128, 64, 4, 40, 40, (8, 8)),
    (64, 33, 6, 30, 30, (1, 1)), (32, 45, 4, 30, 42, (3, 2)),           # pooled planes and images of odd size: deltas and codes begin on any byte
])
@pytest.mark.parametrize("inner", [False, True])
def test_gradient_through_a_pool(cin, cout, batch, h, w, grid, inner):
    """The filter hands channels of x on, and the four pixels of a window differ: the winners are those of x."""
    g = torch.Generator().manual_seed(cin + w)
    place = torch.rand((batch, cin, h // 2, w // 2, 4), generator=g).argsort(-1).reshape(batch, cin, h // 2, w // 2, 2, 2).permute(0, 1, 2, 4, 3, 5).reshape(batch, cin, h, w)
    x = (4 * torch.randint(-2, 2, (batch, cin, h, w), generator=g) + place).bfloat16()         # (-8 .. 7)
    dy = _whole((batch, cout, h // 2, w // 2), 2, g)
    wt = torch.zeros(cout, cin, 3, 3)
    wt[range(cout), [c % cin for c in range(cout)], 1, 1] = 1.0
    layers, ws, at = (conv(cin, cout, 3, slope=1.0), pool(cout)), [wt.bfloat16().cuda(), None], 0
    if inner:
        one = torch.zeros(cin, cin, 1, 1)
        one[range(cin), range(cin)] = 1.0
        layers, ws, at = (conv(cin, cin, 1, slope=1.0),) + layers, [one.bfloat16().cuda()] + ws, cin * cin
    got, kernel = _gradients(layers, batch, h, w, grid, x, ws, dy, at)
    z = x.double()[:, [c % cin for c in range(cout)]]
    cand = z.reshape(batch, cout, h // 2, 2, w // 2, 2).permute(0, 1, 2, 4, 3, 5).reshape(batch, cout, h // 2, w // 2, 4)
    dz = torch.zeros_like(cand).scatter_(-1, cand.argmax(-1, keepdim=True), dy.double()[..., None])
    dz = dz.reshape(batch, cout, h // 2, w // 2, 2, 2).permute(0, 1, 2, 4, 3, 5).reshape(batch, cout, h, w)
    want = _sums(dz, x.double())
    assert kernel == ["k_wgrad_mfma16<%d, 1, %s, true>" % (1 if cin <= 32 else 2, "true" if inner else "false")]
    for v in got:
        assert torch.equal(v.reshape(want.shape), want)
