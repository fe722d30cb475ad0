"""Sums of a layer's shares and of the stacks' gradients: the latter's fixed tree of pairs, bit for bit, around the groups of 8 and 64
stacks and the number of parameters at which another kernel takes over."""
import numpy as np
import pytest
import torch

from ftp_synth.configs import Config, conv
from tests import parity as P

pytestmark = pytest.mark.gpu


def _pairs(v):
    while len(v) > 1:
        v = [v[i] + v[i + 1] if i + 1 < len(v) else v[i] for i in range(0, len(v), 2)]
    return v[0]


@pytest.mark.parametrize("grid", [(1, 1), (2, 4), (3, 3), (4, 4), (7, 9), (8, 8), (5, 13), (8, 9), (11, 12), (16, 16)])
@pytest.mark.parametrize("cin,cout", [(3, 4), (3, 5), (4, 36), (64, 455), (64, 456)])     # 65520 and 65664 groups of 4 parameters
def test_tree_of_pairs(grid, cin, cout):
    from paper_2409_09083_amd.harness import Session
    s = Session((conv(cin, cout),), 1, cin, 32, 32, grid, (1,), "f32")
    g = torch.Generator(device="cuda").manual_seed(3)
    s.partials.copy_(torch.randn(s.partials.shape, generator=g, device="cuda"))
    s.reduce()
    torch.cuda.synchronize()
    want = _pairs(list(s.partials.cpu().numpy()))
    got = s.wgrad.cpu().numpy()
    s.close()
    assert np.array_equal(got, want)


@pytest.mark.parametrize("k,cin,cout,h,w,grid", [
    (3, 3, 4, 416, 416, (1, 1)),                  # 108 parameters: fewer than a workgroup's, 100 shares and more
    (3, 3, 16, 203, 187, (1, 1)),                 # 432: the last workgroup not full
    (3, 3, 5, 200, 200, (1, 1)),                  # 135: no multiple of 4, the other kernel
    (3, 4, 33, 200, 200, (3, 3)),
    (3, 16, 32, 208, 208, (1, 1)),
    (1, 64, 64, 104, 104, (1, 1)),
])
@pytest.mark.parametrize("has_bias", [False, True])
def test_shares_of_a_layer(k, cin, cout, h, w, grid, has_bias):
    """The layer's gradient against sums in 64 bits (no kinks: slope 1)."""
    s = P.make_session(Config("shares", 1, cin, h, w, (conv(cin, cout, k, slope=1.0),), grid, (1,), "f32"), 1, has_bias)
    g = torch.Generator(device="cuda").manual_seed(5)
    s.x.copy_(torch.randn(s.x.shape, generator=g, device="cuda"))
    s.dy.copy_(torch.randn(s.dy.shape, generator=g, device="cuda"))
    s.weights = [torch.randn((cout, cin, k, k), generator=g, device="cuda")]
    if has_bias:
        s.biases = [torch.zeros(cout, device="cuda")]
    s.forward(); s.backward(); s.reduce()
    torch.cuda.synchronize()
    got = s.wgrad.cpu().double().numpy()
    x, dy = s.x.cpu().double(), s.dy.cpu().double()
    s.close()
    xp = torch.nn.functional.pad(x, [k // 2] * 4)
    rows = [(dy[0] * xp[0, c, a:a + h, b:b + w]).sum((1, 2)) for c in range(cin) for a in range(k) for b in range(k)]
    want = torch.stack(rows, 1).reshape(-1).numpy()
    n = len(want)
    assert np.max(np.abs(got[:n] - want)) <= P.TOL_GRAD_F32 * np.max(np.abs(want))
    if has_bias:
        db = dy.sum((0, 2, 3)).numpy()
        assert np.max(np.abs(got[n:n + cout] - db)) <= P.TOL_GRAD_F32 * np.max(np.abs(db))
