"""Maps of three columns and millions of rows, whose pixels the direct kernels count by rows: beyond 2^24 pixels a reciprocal alone no longer tells the row.
Whole numbers, so that all sums are exact."""
import pytest
import torch

from ftp_synth.configs import conv, pool
from paper_2409_09083_amd import binding as B

pytestmark = pytest.mark.gpu


def _step(layers, h, w, weights):
    from paper_2409_09083_amd.harness import Session
    s = Session(layers, 1, layers[0].cin, h, w, (1, 1), (1,), "f32")
    g = torch.Generator(device="cuda").manual_seed(h)
    s.x.copy_(torch.randint(-1, 2, s.x.shape, generator=g, device="cuda"))
    s.dy.copy_(torch.randint(-1, 2, s.dy.shape, generator=g, device="cuda"))
    s.weights = weights
    B.ftp_profile(s.plan, 1)
    s.forward(); s.backward()
    if s.n_params:
        s.reduce()
    torch.cuda.synchronize()
    return s, {r["pass"]: r["kernel"].split("<")[0] for r in B.ftp_profile_read(s.plan)}


def test_pool():
    h, w = 12_700_000, 6
    s, kernels = _step((pool(1),), h, w, [None])
    assert kernels["pool_fwd"] == "k_pool_fwd" and kernels["pool_bwd"] == "k_pool_bwd"
    windows = s.x.view(h // 2, 2, w // 2, 2).permute(0, 2, 1, 3).reshape(h // 2, w // 2, 4)
    first = (windows == windows.amax(-1, keepdim=True)).int().argmax(-1, keepdim=True)            # (the first of equal ones wins)
    assert torch.equal(s.y[0, 0], windows.amax(-1))
    want = torch.zeros_like(windows).scatter_(-1, first, s.dy[0, 0][..., None])
    got = s.dx.view(h // 2, 2, w // 2, 2).permute(0, 2, 1, 3).reshape(h // 2, w // 2, 4)
    assert torch.equal(got, want)
    s.close()


def test_convolution():
    h, w = 6_400_000, 3
    wt = torch.tensor([[1.0, 0.0, -1.0], [2.0, 1.0, 0.0], [0.0, -1.0, 1.0]], device="cuda").view(1, 1, 3, 3)
    big = torch.zeros(1, 1, 5, 5, device="cuda")
    big[:, :, 1:4, 1:4] = wt
    s, kernels = _step((conv(1, 1, 5, slope=1.0),), h, w, [big])
    assert kernels["conv_bwd_data"] == "k_conv_bwd_data_direct"
    pad = lambda t: torch.nn.functional.pad(t[0, 0], (1, 1, 1, 1))
    xp, dp = pad(s.x), pad(s.dy)
    y, dx = torch.zeros_like(s.x[0, 0]), torch.zeros_like(s.x[0, 0])
    for a in range(3):
        for b in range(3):
            y += wt[0, 0, a, b] * xp[a:a + h, b:b + w]
            dx += wt[0, 0, a, b] * dp[2 - a:2 - a + h, 2 - b:2 - b + w]
    assert torch.equal(s.y[0, 0], y) and torch.equal(s.dx[0, 0], dx)
    xp = torch.nn.functional.pad(s.x[0, 0], (2, 2, 2, 2)).double()
    d = s.dy[0, 0].double()
    want = torch.stack([(d * xp[a:a + h, b:b + w]).sum() for a in range(5) for b in range(5)])
    assert torch.equal(s.wgrad.double(), want)
    s.close()
