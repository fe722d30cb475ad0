"""fp32 forward pass of launches that do not fill the chip: the same bits as in a launch of many images, which takes the other kernel - remainders of
channels and stages, rows of every alignment, pools, biases, the caller's buffer and the workspace as input."""
import pytest
import torch

from ftp_synth.configs import conv, pool

pytestmark = pytest.mark.gpu


def _forward(layers, x, ws, bs, grid):
    from paper_2409_09083_amd.harness import Session
    b, c, h, w = x.shape
    s = Session(layers, b, c, h, w, grid, (len(layers),), "f32")
    s.x.copy_(x)
    s.weights = ws
    if any(t is not None for t in bs):
        s.biases = bs
    s.forward()
    torch.cuda.synchronize()
    y = s.y.clone()
    s.close()
    return y


@pytest.mark.parametrize("k,cin,cout,h,w,grid,pooled,inner", [
    (3, 8, 16, 9, 7, (1, 1), False, False),       # fewer stages than are in flight
    (3, 12, 20, 33, 21, (2, 3), False, True),
    (3, 20, 36, 77, 53, (3, 5), False, True),     # the last stage and block are not full
    (3, 64, 96, 24, 34, (2, 2), True, True),
    (3, 40, 16, 34, 70, (1, 1), True, False),     # rows of windows wider than a tile
    (3, 128, 32, 5, 64, (1, 1), False, True),
    (1, 64, 32, 13, 66, (1, 2), False, True),
    (1, 72, 40, 10, 18, (2, 2), True, False),
    (1, 136, 100, 7, 9, (1, 1), False, True),
])
def test_an_image_alone_and_among_many(k, cin, cout, h, w, grid, pooled, inner):
    n = 48
    g = torch.Generator().manual_seed(h * w)
    first = 8 if inner else cin
    x = torch.randn(n, first, h, w, generator=g)
    layers = (conv(first, cin, 1),) if inner else ()
    layers += (conv(cin, cout, k),) + ((pool(cout),) if pooled else ())
    ws = [None if l.kind else (torch.randn(l.cout, l.cin, l.k, l.k, generator=g) / (l.k * l.cin ** 0.5)).cuda() for l in layers]
    bs = []
    for l in layers:
        if l.kind == 0 and l.cout == cout:
            object.__setattr__(l, "has_bias", 1)
            bs.append(torch.randn(cout, generator=g).cuda())
        else:
            bs.append(None)
    many = _forward(layers, x, ws, bs, grid)
    for i in (0, n - 1):
        assert torch.equal(_forward(layers, x[i:i + 1], ws, bs, grid)[0], many[i])
