"""Filter and bias gradients of layers that read the caller's input directly, are narrower than a matrix-core block, or have a
bias: every such gradient against the oracle (sizes large enough for the matrix-core kernels, see wgrad_wide_enough)."""
import pytest

from ftp_synth.configs import Config, conv, pool
from tests import parity as P

pytestmark = pytest.mark.gpu

_NETS = {
    "pooled": ((conv(32, 64), pool(64)), 48, 64),
    "plain": ((conv(40, 48), conv(48, 24)), 30, 46),
    "narrow": ((conv(16, 24), conv(24, 12), conv(12, 8)), 66, 70),
    # odd strides between channels and between images: rows of 16-bit maps that start between dwords
    "oddchannels": ((conv(3, 9), conv(9, 16)), 33, 45),
    "oddpool": ((conv(3, 8), conv(8, 9), pool(9)), 66, 70),
    "oddcaller": ((conv(72, 16, 1), conv(16, 32)), 31, 31),
    "oddwidth": ((conv(16, 40), conv(40, 32)), 33, 45),
    "other": ((conv(24, 20, 5), conv(20, 12, 1), conv(12, 16, 3, stride=2)), 62, 58),
}


@pytest.mark.parametrize("net", sorted(_NETS))
@pytest.mark.parametrize("dtype,bias", [("bf16", False), ("f32", False), ("f32", True), ("bf16", True)])
@pytest.mark.parametrize("grid", [(1, 1), (2, 3)])
def test_gradients(oracle, net, dtype, bias, grid):
    layers, h, w = _NETS[net]
    P.check_case(oracle, Config("routes_" + net, 3, layers[0].cin, h, w, layers, grid, (len(layers),), dtype), has_bias=bias)


def _kernels(layers, batch, h, w, grid, dtype, passes, has_bias=False):
    """Kernels that the first layer's launches of these passes ran (a step on random values)."""
    import torch
    from paper_2409_09083_amd import binding as B
    from paper_2409_09083_amd.harness import Session
    s = Session([P._BiasLayer(ly) for ly in layers] if has_bias else layers, batch, layers[0].cin, h, w, grid, (len(layers),), dtype=dtype)
    s.x.uniform_(0, 1)
    s.dy.normal_()
    s.weights = [torch.randn((ly.cout, ly.cin, ly.k, ly.k), device="cuda").to(s.x.dtype) / 20 for ly in layers]
    s.biases = [torch.zeros(ly.cout, device="cuda").to(s.x.dtype) for ly in layers] if has_bias else None
    B.ftp_profile(s.plan, 1)
    s.step()
    torch.cuda.synchronize()
    names = {r["kernel"].split("<")[0] for r in B.ftp_profile_read(s.plan) if r["pass"] in passes and r["layer"] == 0}
    s.close()
    return names


@pytest.mark.parametrize("layer,small,large", [
    (conv(16, 32), (1, 52, (2, 2)), (8, 52, (1, 1))), (conv(64, 64), (1, 13, (1, 1)), (1, 26, (2, 2))), (conv(32, 32, 1), (8, 13, (1, 1)), (16, 104, (1, 1))),
    (conv(3, 16), (1, 52, (2, 2)), (8, 52, (1, 1))), (conv(16, 32, 5), (1, 13, (1, 1)), (8, 52, (1, 1)))])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_small_gradients_with_a_bias_stay_one_launch(layer, small, large, dtype):
    """(sizes at which either kernel is clearly the faster one)"""
    wgrad = lambda size: _kernels((layer,), size[0], size[1], size[1], size[2], dtype, ("wgrad", "wgrad_sum"), has_bias=True)
    assert wgrad(small) == {"k_wgrad_direct"}
    assert "k_wgrad_direct" not in wgrad(large)


@pytest.mark.parametrize("layer,size,dtype,direct", [
    (conv(8, 16, 1), (16, 128, (2, 2)), "f32", True), (conv(8, 32, 1), (16, 128, (2, 2)), "f32", False), (conv(8, 8, 1), (16, 128, (2, 2)), "bf16", True),
    (conv(8, 8), (16, 128, (2, 2)), "f32", False), (conv(8, 16), (1, 32, (1, 1)), "f32", False),
    (conv(8, 8, 3, stride=2), (16, 128, (2, 2)), "f32", True), (conv(12, 16, 3, stride=2), (16, 128, (2, 2)), "f32", False), (conv(8, 12, 3, stride=2), (1, 128, (2, 2)), "f32", False),
    (conv(8, 16, 1, stride=2), (1, 32, (1, 1)), "f32", True), (conv(8, 48, 1, stride=2), (1, 32, (1, 1)), "f32", False)])
def test_narrow_deltas_take_the_faster_kernel(layer, size, dtype, direct):
    batch, hw, grid = size
    names = _kernels((layer,), batch, hw, hw, grid, dtype, ("conv_bwd_data",))
    assert ("k_conv_bwd_data_direct" in names) == direct, names


@pytest.mark.parametrize("layer,size,direct", [(conv(48, 3, 3, stride=2), (16, 128, (4, 3)), True), (conv(48, 24, 3, stride=2), (16, 128, (4, 3)), False), (conv(208, 16), (4, 104, (1, 1)), False)])
def test_narrow_gradients_take_the_faster_kernel(layer, size, direct):
    batch, hw, grid = size
    assert ("k_wgrad_direct" in _kernels((layer,), batch, hw, hw, grid, "f32", ("wgrad",))) == direct


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("layers,batch,h,w,grid", [((conv(16, 40, slope=1.0),), 5, 97, 131, (1, 1)), ((conv(16, 40, slope=1.0), pool(40)), 5, 98, 130, (1, 1)),
                                                   ((conv(48, 64, 1, slope=1.0),), 3, 33, 45, (2, 3)), ((conv(64, 64, slope=1.0),), 1, 31, 29, (1, 1))])
def test_bias_gradients_against_64_bits(layers, batch, h, w, grid, dtype):
    """Sums of one workgroup a channel and stack: a few hundred deltas, and more than its threads take in one go."""
    import torch
    from paper_2409_09083_amd.harness import Session
    s = Session([P._BiasLayer(layers[0])] + list(layers[1:]), batch, layers[0].cin, h, w, grid, (len(layers),), dtype=dtype)
    g = torch.Generator(device="cuda").manual_seed(8)
    s.x.uniform_(0, 1, generator=g)
    s.dy.normal_(generator=g)
    s.weights = [torch.randn(tuple((layers[0].cout, layers[0].cin, layers[0].k, layers[0].k)), device="cuda", generator=g).to(s.x.dtype) / 20] + [None] * (len(layers) - 1)
    s.biases = [torch.zeros(layers[0].cout, device="cuda").to(s.x.dtype)] + [None] * (len(layers) - 1)
    s.step()
    torch.cuda.synchronize()
    got = s.wgrad[-layers[0].cout:].double()
    ref, mag = s.dy.double().sum((0, 2, 3)), s.dy.double().abs().sum((0, 2, 3))
    # (fp32 sums: a rounding of 2^-24 of the magnitudes per addition of a thread, 64 at most here, of the tree and the last sum)
    assert bool(((got - ref).abs() <= 100 * 2.0 ** -24 * mag).all())
    s.close()


@pytest.mark.parametrize("cin,cout,batch,h,w,grid,kernel", [
    (6, 24, 24, 140, 138, (2, 2), "k_wgrad_mfma_thin"), (6, 24, 23, 140, 138, (2, 2), "k_wgrad_mfma"),          # as many pixels and fewer
    (6, 24, 22, 100, 208, (1, 2), "k_wgrad_mfma_thin"), (6, 24, 22, 100, 210, (1, 2), "k_wgrad_mfma"),          # the widest rows
    (7, 32, 8, 200, 288, (3, 3), "k_wgrad_mfma_thin"), (7, 33, 8, 200, 288, (3, 3), "k_wgrad_mfma"),
    (8, 16, 24, 140, 138, (2, 2), "k_wgrad_mfma_thin"), (8, 17, 24, 140, 138, (2, 2), "k_wgrad_mfma"),
    (5, 16, 16, 170, 170, (4, 4), "k_wgrad_mfma_thin"), (7, 16, 16, 170, 170, (4, 4), "k_wgrad_mfma"),          # rows of 42 and 43
])
def test_narrow_1x1_layers(cin, cout, batch, h, w, grid, kernel):
    """The kernel that each side of the rule's lines takes; whole numbers, so that the sums are exact in any order."""
    _narrow((conv(cin, cout, 1, slope=1.0),), batch, h, w, grid, "f32", kernel)


@pytest.mark.parametrize("dtype,cin,cout,batch,h,w,grid,kernel", [
    ("f32", 5, 32, 4, 300, 208, (3, 8), "k_wgrad_mfma_thin"), ("f32", 5, 33, 4, 300, 208, (3, 8), "k_wgrad_mfma"),             # rows of 26
    ("f32", 12, 20, 4, 250, 240, (3, 10), "k_wgrad_mfma"), ("f32", 12, 20, 4, 250, 244, (3, 9), "k_wgrad_mfma_thin"),            # rows of 24, and 26 and 28
    ("f32", 13, 20, 4, 250, 244, (3, 9), "k_wgrad_mfma"), ("f32", 12, 20, 3, 250, 244, (3, 9), "k_wgrad_mfma"),
    ("bf16", 6, 28, 6, 248, 204, (2, 6), "k_wgrad_mfma_thin"), ("bf16", 6, 28, 6, 248, 204, (2, 7), "k_wgrad_mfma"),           # rows of 34, and 28 and 30
    ("bf16", 8, 20, 6, 248, 204, (2, 4), "k_wgrad_mfma_thin"), ("bf16", 8, 20, 5, 248, 204, (2, 4), "k_wgrad_mfma"),
    ("bf16", 9, 20, 8, 248, 240, (2, 6), "k_wgrad_mfma_thin"), ("bf16", 9, 20, 8, 248, 240, (2, 7), "k_wgrad_mfma"),           # rows of 40, and 34 and 36
    ("bf16", 12, 32, 8, 300, 200, (1, 2), "k_wgrad_mfma_thin"), ("bf16", 12, 32, 7, 300, 200, (1, 2), "k_wgrad_mfma"),
])
def test_narrow_1x1_layers_with_a_pool(dtype, cin, cout, batch, h, w, grid, kernel):
    """The filter hands channels of x on, and the four pixels of a window differ: the winners are those of x."""
    _narrow((conv(cin, cout, 1, slope=1.0), pool(cout)), batch, h, w, grid, dtype, kernel)


def _narrow(layers, batch, h, w, grid, dtype, kernel):
    import torch
    from paper_2409_09083_amd import binding as B
    from paper_2409_09083_amd.harness import Session
    cin, cout, pooled = layers[0].cin, layers[0].cout, len(layers) > 1
    g = torch.Generator(device="cuda").manual_seed(cin)
    s = Session(layers, batch, cin, h, w, grid, (len(layers),), dtype)
    one = [[c % cin] for c in range(cout)]
    if pooled:
        place = torch.rand((batch, cin, h // 2, w // 2, 4), generator=g, device="cuda").argsort(-1)
        place = place.reshape(batch, cin, h // 2, w // 2, 2, 2).permute(0, 1, 2, 4, 3, 5).reshape(s.x.shape)
        s.x.copy_(4 * torch.randint(-2, 2, s.x.shape, generator=g, device="cuda") + place)          # (-8 .. 7)
    else:
        s.x.copy_(torch.randint(-4, 5, s.x.shape, generator=g, device="cuda"))
    s.dy.copy_(torch.randint(-2, 3, s.dy.shape, generator=g, device="cuda"))
    wt = torch.zeros(cout, cin, device="cuda").scatter_(1, torch.tensor(one, device="cuda"), 1.0).view(cout, cin, 1, 1).to(s.tdtype)
    s.weights = [wt] + [None] * pooled
    B.ftp_profile(s.plan, 1)
    s.step()
    torch.cuda.synchronize()
    assert [r["kernel"].split("<")[0] for r in B.ftp_profile_read(s.plan) if r["pass"] == "wgrad"] == [kernel]
    got, x, dz = s.wgrad.double().reshape(cout, cin), s.x.double(), s.dy.double()
    s.close()
    if pooled:
        z = x[:, [c[0] for c in one]].reshape(batch, cout, h // 2, 2, w // 2, 2).permute(0, 1, 2, 4, 3, 5).reshape(batch, cout, h // 2, w // 2, 4)
        dz = torch.zeros_like(z).scatter_(-1, z.argmax(-1, keepdim=True), dz[..., None])
        dz = dz.reshape(batch, cout, h // 2, w // 2, 2, 2).permute(0, 1, 2, 4, 3, 5).reshape(batch, cout, h, w)
    assert 8 * batch * h * w < 2 ** 24
    x, dz = x.transpose(0, 1).reshape(cin, -1), dz.transpose(0, 1).reshape(cout, -1)
    assert torch.equal(got, dz @ x.T)
