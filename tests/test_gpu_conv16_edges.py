"""16-bit stride-1 1x1 / 3x3 convolutions at the edges of their stages (reduction channels from one group of 8 to several stages and
a remainder), small launches, maps in the caller's buffer whose rows, channels and images start between dwords."""
import pytest
import torch

from ftp_synth.configs import Config, conv, pool
from tests import parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 3])
@pytest.mark.parametrize("cin", [8, 9, 17, 25, 33, 40, 56, 65, 72, 100, 129])
@pytest.mark.parametrize("h,w,pooled", [(13, 9, False), (14, 22, True)])
def test_channels(oracle, k, cin, h, w, pooled):
    layers = (conv(cin, 36, k),) + ((pool(36),) if pooled else ()) + (conv(36, cin, k),)
    P.check_case(oracle, Config("edges16", 3, cin, h, w, layers, (2, 1), (len(layers),), "bf16"))


@pytest.mark.parametrize("k", [1, 3])
@pytest.mark.parametrize("cin,h,w,batch", [(9, 31, 13, 3), (24, 15, 11, 4), (17, 7, 5, 5), (40, 40, 44, 2), (64, 75, 75, 16)])
@pytest.mark.parametrize("offset", [0, 1, 2, 3])
def test_caller_buffers_that_start_anywhere(k, cin, h, w, batch, offset):
    """The same image, `offset` elements into a buffer: the same bits, nothing read beside it is used (it is NaN there)."""
    from paper_2409_09083_amd.harness import Session
    s = Session((conv(cin, 48, k), conv(48, 16, k)), batch, cin, h, w, (2, 1), (2,), dtype="bf16")
    g = torch.Generator(device="cuda").manual_seed(7)
    x = torch.empty(s.in_shape, device="cuda").normal_(generator=g).bfloat16()
    s.weights = [(torch.empty((o, i, k, k), device="cuda").normal_(generator=g) / 8).bfloat16() for i, o in ((cin, 48), (48, 16))]
    s.dy.normal_(generator=g)
    s.x.copy_(x)
    s.step()
    ref = [t.clone() for t in (s.y, s.dx, s.wgrad)]
    n = x.numel()
    buf = torch.full((n + 64,), float("nan"), dtype=torch.bfloat16, device="cuda")
    buf[16 + offset:16 + offset + n] = x.reshape(-1)
    s.x = buf[16 + offset:16 + offset + n].view(s.in_shape)
    s.workspace.fill_(0xFF)
    s.step()
    torch.cuda.synchronize()
    assert torch.equal(s.y, ref[0]) and torch.equal(s.dx, ref[1])
    # (the filter gradient of a buffer that is not on a dword takes another kernel, in another order of sums)
    assert float((s.wgrad - ref[2]).norm() / ref[2].norm()) < 1e-5
    s.close()


def test_caller_buffers_beyond_2_gib():
    """Maps that begin between dwords in a buffer of more than 2 GiB: an image has the bits that it has alone, the first ones and the last."""
    from paper_2409_09083_amd.harness import Session
    g = torch.Generator(device="cuda").manual_seed(12)
    x = torch.empty((1, 16, 513, 511), device="cuda").normal_(generator=g).bfloat16()
    w = (torch.empty((64, 16, 3, 3), device="cuda").normal_(generator=g) / 12).bfloat16()
    out = []
    for batch in (1, 260):
        s = Session((conv(16, 64),), batch, 16, 513, 511, (1, 2), (1,), dtype="bf16")
        s.x.copy_(x.expand(s.in_shape))
        s.weights = [w]
        s.forward()
        torch.cuda.synchronize()
        out.append(s.y)
        s.close()
    assert 2 * 260 * x.numel() > 2 ** 31
    assert all(torch.equal(out[1][n], out[0][0]) for n in range(260))
