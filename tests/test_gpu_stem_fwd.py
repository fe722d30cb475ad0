"""First layers (at most 4 input channels) against the oracle: tiles of one and several columns and rows, the last ones partly
filled, runs of tiles that a workgroup takes one after the other, channel counts around blocks of 16 and 32, biases, every filter."""
import pytest

from ftp_synth.configs import Config, conv, pool
from tests import parity as P

pytestmark = pytest.mark.gpu


def _biased(ly):
    object.__setattr__(ly, "has_bias", 1)
    return ly


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("cin,cout,batch,h,w,grid", [
    (3, 8, 1, 6, 6, (1, 1)), (1, 17, 2, 34, 66, (1, 1)), (4, 33, 1, 70, 130, (2, 2)), (3, 64, 3, 36, 10, (3, 1)),
    (3, 32, 64, 136, 32, (2, 2)), (2, 16, 64, 72, 48, (4, 4))])
def test_pooled(oracle, dtype, cin, cout, batch, h, w, grid):
    P.check_case(oracle, Config("stem", batch, cin, h, w, (conv(cin, cout), pool(cout)), grid, (2,), dtype))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("k,stride,cin,cout,batch,h,w,grid", [
    (3, 1, 3, 8, 1, 5, 7, (1, 1)), (3, 1, 4, 40, 2, 33, 65, (2, 1)), (3, 1, 3, 16, 64, 76, 40, (4, 4)), (3, 2, 2, 20, 2, 35, 67, (1, 2)),
    (5, 1, 3, 24, 1, 18, 34, (1, 1)), (5, 2, 4, 16, 1, 37, 41, (2, 2)), (7, 1, 1, 48, 1, 17, 33, (1, 1)), (7, 2, 3, 64, 2, 67, 131, (2, 1)),
    (7, 2, 4, 72, 1, 65, 67, (1, 1)), (7, 2, 4, 16, 1, 32, 32, (1, 1)), (7, 2, 4, 20, 2, 64, 30, (2, 1)), (1, 2, 3, 36, 2, 31, 70, (1, 3))])
def test_unpooled(oracle, dtype, k, stride, cin, cout, batch, h, w, grid):
    P.check_case(oracle, Config("stem", batch, cin, h, w, (conv(cin, cout, k, stride=stride),), grid, (1,), dtype))


@pytest.mark.parametrize("slope", [0.0, 1.0, 1.5])
def test_slopes_and_bias(slope):
    """Slopes outside (0, 1) and a bias take the general epilogue: values against 64 bits."""
    import torch
    from paper_2409_09083_amd.harness import Session
    g = torch.Generator().manual_seed(3)
    s = Session((_biased(conv(3, 20, slope=slope)), pool(20)), 2, 3, 38, 44, (1, 2), (2,))
    x, w, b = torch.randn(s.in_shape, generator=g), torch.randn((20, 3, 3, 3), generator=g) / 5, torch.randn(20, generator=g)
    s.load(x=x.numpy(), weights=[w.numpy(), None], biases=[b.numpy(), None])
    s.forward()
    z = torch.nn.functional.conv2d(x.double(), w.double(), b.double(), padding=1)
    ref = torch.nn.functional.max_pool2d(torch.where(z > 0, z, z * slope), 2)
    # (27 products and their sums, each rounded to 24 bits)
    assert float((s.y.cpu().double() - ref).abs().max() / ref.abs().max()) < 28 * 2.0 ** -24
    s.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("h,w,cout,grid,slope", [(13, 13, 12, (1, 1), 0.1), (16, 24, 37, (2, 2), 0.1), (9, 31, 4, (1, 3), 1.0), (32, 40, 64, (2, 1), 0.5)])
def test_step_whose_launches_carry_the_filter_relayout(oracle, dtype, h, w, cout, grid, slope):
    """The first layer's forward pass and the scaling of dy (single pixels and groups, channel counts around groups of 4) relay the
    filters of the layers behind: forward, deltas and gradients of a network of two, and of one with more jobs than travel along."""
    def net(n):
        ls = [conv(3, 16)]
        for i in range(n):
            ls.append(conv(16 if i == 0 else cout, cout, slope=slope if i == n - 1 else 0.1))
        return tuple(ls)
    P.check_case(oracle, Config("carry", 2, 3, h, w, net(1), grid, (2,), dtype))
    P.check_case(oracle, Config("carry9", 1, 3, h, w, net(10), (1, 1), (4, 11), dtype))


@pytest.mark.parametrize("cin,cout", [(36, 72), (33, 65)])
def test_bias_sums_travel_with_the_shares(cin, cout):
    """A small layer with a bias whose gradient comes in shares, 4 and 1 parameters a thread: the gradient against 64 bits."""
    import torch
    from paper_2409_09083_amd.harness import Session
    g = torch.Generator().manual_seed(4)
    s = Session((_biased(conv(cin, cout, slope=1.0)),), 3, cin, 44, 40, (2, 1), (1,))
    x, w, b = torch.randn(s.in_shape, generator=g), torch.randn((cout, cin, 3, 3), generator=g) / 18, torch.randn(cout, generator=g)
    dy = torch.randn(tuple(s.dy.shape), generator=g)
    s.load(x=x.numpy(), weights=[w.numpy()], biases=[b.numpy()], dy=dy.numpy())
    s.step()
    w64, b64 = w.double().requires_grad_(True), b.double().requires_grad_(True)
    torch.nn.functional.conv2d(x.double(), w64, b64, padding=1).backward(dy.double())
    got, n = s.wgrad.cpu().double(), w.numel()
    # (5280 products of normal numbers: sums of about 73, every partial sum rounded to 24 bits)
    for a, ref in ((got[:n], w64.grad.reshape(-1)), (got[n:], b64.grad)):
        assert float((a - ref).abs().max() / ref.abs().max()) < 1e-5
    s.close()


def _one_layer(k, stride, cin, cout, batch, h, w, grid, dtype, pooled, x, weights):
    """y, signs, decision codes (all of image 0) and the kernel of a first layer's forward pass over copies of one image."""
    import torch
    from paper_2409_09083_amd import binding as B
    from paper_2409_09083_amd.harness import Session
    s = Session((conv(cin, cout, k, stride=stride),) + ((pool(cout),) if pooled else ()), batch, cin, h, w, grid, (2 if pooled else 1,), dtype)
    s.x.copy_(x.expand(s.in_shape))
    s.weights = [weights] + [None] * pooled
    B.ftp_profile(s.plan, 1)
    s.forward()
    torch.cuda.synchronize()
    names = {r["kernel"].split("<")[0] for r in B.ftp_profile_read(s.plan)}
    last = 2 if pooled else 1
    out = [s.y[0].clone(), s._buffer(last, B.FTP_BUF_SIGN)[0][0].clone()]
    if pooled:
        out.append(s._buffer(last, B.FTP_BUF_MASK)[0][0].clone())
    s.close()
    return out, names


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("k,stride,cin,cout,batch,h,w,grid,pooled", [
    (3, 1, 3, 8, 10, 128, 130, (2, 2), True), (3, 1, 4, 9, 70, 124, 128, (1, 1), True), (3, 1, 3, 20, 20, 129, 131, (1, 3), False), (3, 1, 2, 37, 20, 127, 128, (1, 1), False),
    (5, 1, 3, 4, 5, 131, 130, (2, 1), False), (7, 1, 1, 4, 5, 128, 133, (1, 1), False), (3, 2, 3, 8, 124, 129, 130, (1, 2), False)])
def test_few_channels_of_large_launches_take_the_vector_alu(dtype, k, stride, cin, cout, batch, h, w, grid, pooled):
    """The two kernels add in the same order: an image alone and among many has the same bits."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(7)
    x = torch.randn((1, cin, h, w), device="cuda", generator=g)
    weights = (torch.randn((cout, cin, k, k), device="cuda", generator=g) / (k * cin ** 0.5)).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    alone, small = _one_layer(k, stride, cin, cout, 1, h, w, grid, dtype, pooled, x, weights)
    many, large = _one_layer(k, stride, cin, cout, batch, h, w, grid, dtype, pooled, x, weights)
    assert small == {"k_conv_fwd_stem"} and large == {"k_conv_fwd_thin" if k == 3 and stride == 1 else "k_conv_fwd_thin_gen"}
    for a, b in zip(alone, many):
        assert torch.equal(a, b)


def test_maps_beyond_the_matrix_kernel_offsets():
    """A map of more than 2 GB over all channels: the vector ALU's kernel, checked at two corners against 64 bits."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(9)
    n = 2304
    x, w = torch.randn((1, 3, n, n), device="cuda", generator=g), torch.randn((64, 3, 3, 3), device="cuda", generator=g) / 5
    (y, _), names = _one_layer(3, 1, 3, 64, 1, n, n, (1, 1), "f32", False, x, w)
    assert names == {"k_conv_fwd_thin"}
    z = lambda part: torch.nn.functional.conv2d(part.cpu().double(), w.cpu().double(), padding=1)
    for got, ref in ((y[:, :40, :40], z(x[:, :, :41, :41])[0, :, :40, :40]), (y[:, -40:, -40:], z(x[:, :, -41:, -41:])[0, :, 1:, 1:])):
        ref = torch.where(ref > 0, ref, ref * 0.1)
        # (27 products and their sums, each rounded to 24 bits)
        assert float((got.cpu().double() - ref).abs().max() / ref.abs().max()) < 28 * 2.0 ** -24


@pytest.mark.parametrize("batch,h,w,grid,thin", [(20, 127, 128, (1, 1), False), (20, 127, 129, (1, 1), True), (20, 126, 130, (1, 2), True), (20, 126, 130, (1, 5), False), (2, 127, 129, (1, 1), False)])
def test_16_bit_rows_between_dwords(batch, h, w, grid, thin):
    """Tile columns of 65 pixels (half begin between dwords), of 26 (none do), odd rows; the same bits from either kernel."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(8)
    x, weights = torch.randn((1, 3, h, w), device="cuda", generator=g), (torch.randn((32, 3, 3, 3), device="cuda", generator=g) / 5).to(torch.bfloat16)
    many, names = _one_layer(3, 1, 3, 32, batch, h, w, grid, "bf16", False, x, weights)
    assert names == {"k_conv_fwd_thin" if thin else "k_conv_fwd_stem"}
    alone, names = _one_layer(3, 1, 3, 32, 1, h, w, grid, "bf16", False, x, weights)
    assert names == {"k_conv_fwd_stem"}
    for a, b in zip(alone, many):
        assert torch.equal(a, b)
