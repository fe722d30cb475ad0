"""fp32 delta back-propagation on the bfloat matrix cores (three-way split): single layers against 64-bit sums, at channel
counts and map sizes around the edges of the kernel's groups and tiles; infinities and NaN."""
import numpy as np
import pytest
import torch

from ftp_synth.configs import CONV, conv, pool

pytestmark = pytest.mark.gpu


def _session(layers, batch, h, w, grid, seed):
    from paper_2409_09083_amd.harness import Session
    g = torch.Generator().manual_seed(seed)
    s = Session(layers, batch, layers[0].cin, h, w, grid, (len(layers),))
    x = torch.rand(s.in_shape, generator=g) * 2 - 0.5
    ws = [torch.randn((ly.cout, ly.cin, ly.k, ly.k), generator=g) / np.sqrt(ly.cin * ly.k * ly.k) if ly.kind == CONV else None for ly in layers]
    dy = torch.randn(s.out_shape, generator=g)
    return s, x, ws, dy


def _load(s, x, ws, dy):
    s.x.copy_(x)
    s.dy.copy_(dy)
    s.weights = [None if w is None else w.cuda().contiguous() for w in ws]


def _bound(x, w, ly, op):
    """Elementwise: dropped products (at most 2^-24 of each product) plus one fp32 rounding of a partial sum per 8 reduction
    elements and plane product (each at most 2^-24 of the sum of magnitudes)."""
    mag = op(x.abs().double(), w.abs().double())
    n = 6 * (ly.k * ly.k * ((max(ly.cin, ly.cout) + 7) // 8 + 1)) + 8
    return (n + 1) * 2.0 ** -24 * mag + 1e-30


@pytest.mark.parametrize("cin,cout", [(16, 8), (20, 9), (36, 17), (132, 24), (64, 40)])
@pytest.mark.parametrize("k,stride", [(3, 1), (1, 1), (5, 1), (7, 1), (3, 2)])
def test_single_layer(cin, cout, k, stride):
    ly = conv(cin, cout, k, slope=1.0, stride=stride)
    for i, (batch, h, w, grid) in enumerate([(1, 13, 17, (1, 1)), (3, 31, 22, (2, 3))]):
        s, x, ws, dy = _session((ly,), batch, h, w, grid, 11 + i)
        _load(s, x, ws, dy)
        s.step()
        torch.cuda.synchronize()
        bwd = lambda a, b: torch.nn.grad.conv2d_input(x.shape, b, a, stride=stride, padding=k // 2)
        err = (s.dx.cpu().double() - bwd(dy.double(), ws[0].double())).abs()
        assert bool((err <= _bound(dy, ws[0], ly, bwd)).all()), (batch, float(err.max()))
        s.close()


@pytest.mark.parametrize("pooled", [False, True])
def test_non_finite_deltas_come_out_as_fp32_sums_give_them(pooled):
    layers = (conv(24, 40), pool(40)) if pooled else (conv(24, 40),)
    s, x, ws, dy = _session(layers, 2, 20, 28, (2, 2), 5)
    dy[0, 3, 4, 5] = float("inf")
    dy[0, 9, 8, 11] = float("-inf")
    dy[1, 0, 0, 0] = float("nan")
    dy[1, 7, -1, -1] = 3.4e38                       # above the largest bfloat
    dy[1, 30, 5, 9] = 1e-38
    _load(s, x, ws, dy)
    s.step()
    torch.cuda.synchronize()
    xr = x.clone().requires_grad_(True)
    y = torch.nn.functional.leaky_relu(torch.nn.functional.conv2d(xr, ws[0], padding=1), 0.1)
    if pooled:
        y = torch.nn.functional.max_pool2d(y, 2)
    (ref,) = torch.autograd.grad(y, xr, dy)
    got = s.dx.cpu()
    fin = torch.isfinite(ref)
    assert torch.equal(torch.isfinite(got), fin)
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    assert torch.equal(got[torch.isinf(ref)], ref[torch.isinf(ref)])
    assert float(((got - ref).abs() / (ref.abs() + 1))[fin].max()) < 1e-5
    s.close()


@pytest.mark.parametrize("k,pooled", [(1, False), (3, False), (5, False), (7, False), (1, True), (3, True)])
@pytest.mark.parametrize("cin,cout", [(16, 64), (36, 48), (132, 24)])
def test_no_plane_is_missing(k, pooled, cin, cout):
    """The norm of the error against 64 bits: about 1.4e-7 with all six products (the roundings of the sums); random sums without one
    of the three smallest products are off by 2.4e-6 and more."""
    layers = (conv(cin, cout, k, slope=1.0),) + ((pool(cout),) if pooled else ())
    s, x, ws, dy = _session(layers, 2, 32, 44, (1, 2), 17)
    _load(s, x, ws, dy)
    s.step()
    torch.cuda.synchronize()
    dz = dy.double()
    if pooled:
        y = torch.nn.functional.conv2d(x.double(), ws[0].double(), padding=k // 2)
        _, idx = torch.nn.functional.max_pool2d(y, 2, return_indices=True)
        dz = torch.zeros(2, cout, 32 * 44, dtype=torch.float64).scatter_(2, idx.flatten(2), dz.flatten(2)).reshape(2, cout, 32, 44)
    ref = torch.nn.grad.conv2d_input(x.shape, ws[0].double(), dz, padding=k // 2)
    err = float((s.dx.cpu().double() - ref).norm() / ref.norm())
    assert err < 5e-7
    s.close()
