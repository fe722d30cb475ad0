"""fp32 forward pass of launches that do not fill the chip, the kernel that each side takes named: the same bits - values, winner codes, signs - as in a launch of many images, which takes
the other kernel: remainders of channels and stages, rows of every alignment, pools, biases, the caller's buffer and the workspace as input."""
import pytest
import torch

from ftp_synth.configs import conv, pool
from paper_2409_09083_amd import binding as B

pytestmark = pytest.mark.gpu


def _forward(layers, x, ws, bs, grid, images):
    """y, signs and codes of `images`, and the kernel of the last convolution."""
    from paper_2409_09083_amd.harness import Session
    b, c, h, w = x.shape
    s = Session(layers, b, c, h, w, grid, (len(layers),), "f32")
    s.x.copy_(x)
    s.weights = ws
    if any(t is not None for t in bs):
        s.biases = bs
    s.workspace.zero_()                               # (words and codes of pixels that no stack owns are never written)
    B.ftp_profile(s.plan, 1)
    s.forward()
    torch.cuda.synchronize()
    last = max(i for i, l in enumerate(layers) if l.kind == 0)
    kernel = [r["kernel"] for r in B.ftp_profile_read(s.plan) if r["pass"] == "conv_fwd" and r["layer"] == last]
    maps = [s.y] + [s._buffer(len(layers), which)[0] for which in (B.FTP_BUF_SIGN, B.FTP_BUF_MASK)]
    out = [m[images].clone() for m in maps if m is not None]
    s.close()
    return out, kernel


@pytest.mark.parametrize("k,cin,cout,h,w,grid,pooled,inner,n", [
    (3, 8, 16, 9, 7, (1, 1), False, False, 270),       # fewer stages than are in flight
    (3, 12, 20, 33, 21, (2, 3), False, True, 48),
    (3, 20, 36, 77, 53, (3, 5), False, True, 24),      # the last stage and block are not full
    (3, 64, 96, 24, 34, (2, 2), True, True, 12),
    (3, 40, 16, 34, 70, (1, 1), True, False, 12),      # rows of windows wider than a tile
    (3, 128, 32, 5, 64, (1, 1), False, True, 60),      # 32 stages
    (1, 64, 32, 13, 66, (1, 2), False, True, 48),
    (1, 72, 40, 10, 18, (2, 2), True, False, 48),
    (1, 136, 100, 7, 9, (1, 1), False, True, 80),
])
def test_an_image_alone_and_among_many(k, cin, cout, h, w, grid, pooled, inner, n):
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
    many, other = _forward(layers, x, ws, bs, grid, [0, n - 1])
    assert len(other) == 1 and other[0].startswith("k_conv_mfma_dl<float, %d, " % k)
    assert len(many) == (3 if pooled else 2)
    for j, i in enumerate((0, n - 1)):
        alone, small = _forward(layers, x[i:i + 1], ws, bs, grid, [0])
        assert small == ["k_conv_small<%d, %s, %s>" % (k, "true" if pooled else "false", "true" if inner else "false")]
        assert all(torch.equal(a[0], m[j]) for a, m in zip(alone, many))
