"""Sums of a layer's shares, of whole numbers, and of the stacks' gradients, the kernel named: the latter's fixed tree of pairs, bit for bit, around the groups of 8 and 64
stacks and the number of parameters at which another kernel takes over."""
import numpy as np
import pytest
import torch

from ftp_synth.configs import Config, conv
from paper_2409_09083_amd import binding as B
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
    B.ftp_profile(s.plan, 1)
    s.reduce()
    torch.cuda.synchronize()
    stacks, groups = grid[0] * grid[1], s.n_params / 4
    shared = s.n_params % 4 == 0 and stacks > (8 if groups <= 65536 else 63)
    assert [r["kernel"] for r in B.ftp_profile_read(s.plan)] == ["k_reduce_wgrad_shared" if shared else "k_reduce_wgrad"]
    want = _pairs(list(s.partials.cpu().numpy()))
    got = s.wgrad.cpu().numpy()
    s.close()
    assert np.array_equal(got, want)


@pytest.mark.parametrize("k,cin,cout,h,w,grid,few", [
    (3, 3, 4, 416, 416, (1, 1), True),                  # 108 parameters: fewer than a workgroup's, 100 shares and more
    (3, 3, 16, 203, 187, (1, 1), True),                 # 432: the last workgroup not full
    (3, 3, 5, 200, 200, (1, 1), False),                 # 135: no multiple of 4, the other kernel
    (3, 4, 33, 200, 200, (3, 3), True),
    (3, 16, 32, 208, 208, (1, 1), True),
    (1, 64, 64, 104, 104, (1, 1), True),
])
@pytest.mark.parametrize("has_bias", [False, True])
def test_shares_of_a_layer(k, cin, cout, h, w, grid, few, has_bias):
    """Operands are small whole numbers: the shares' sums are exact in any order, and a share that is missed or doubled shows."""
    s = P.make_session(Config("shares", 1, cin, h, w, (conv(cin, cout, k, slope=1.0),), grid, (1,), "f32"), 1, has_bias)
    g = torch.Generator(device="cuda").manual_seed(5)
    s.x.copy_(torch.randint(-4, 5, s.x.shape, generator=g, device="cuda"))
    s.dy.copy_(torch.randint(-2, 3, s.dy.shape, generator=g, device="cuda"))
    s.weights = [torch.randn((cout, cin, k, k), generator=g, device="cuda")]
    if has_bias:
        s.biases = [torch.zeros(cout, device="cuda")]
    B.ftp_profile(s.plan, 1)
    s.forward(); s.backward(); s.reduce()
    torch.cuda.synchronize()
    kernels = {r["kernel"] for r in B.ftp_profile_read(s.plan)}
    assert ("k_wgrad_shares_few" in kernels, "k_wgrad_splitk_reduce" in kernels) == (few, not few)
    got = s.wgrad.cpu().double().numpy()
    x, dy = s.x.cpu().double(), s.dy.cpu().double()
    s.close()
    assert 8 * h * w < 2 ** 24
    xp = torch.nn.functional.pad(x, [k // 2] * 4)
    rows = [(dy[0] * xp[0, c, a:a + h, b:b + w]).sum((1, 2)) for c in range(cin) for a in range(k) for b in range(k)]
    want = torch.stack(rows, 1).reshape(-1).numpy()
    n = len(want)
    assert np.array_equal(got[:n], want)
    if has_bias:
        assert np.array_equal(got[n:n + cout], dy.sum((0, 2, 3)).numpy())
