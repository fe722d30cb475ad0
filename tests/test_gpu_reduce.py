"""Sum of the stacks' gradients: its fixed tree of pairs, bit for bit, around the groups of 8 and 64 stacks and the number of parameters at which another
kernel takes over."""
import numpy as np
import pytest
import torch

from ftp_synth.configs import conv

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
