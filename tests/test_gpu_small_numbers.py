"""fp32 gradients of very small numbers: deltas, filters and inputs down to the smallest fp32 numbers keep all their bits."""
import pytest
import torch

from ftp_synth.configs import conv, pool

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,pooled", [(3, False), (3, True), (1, False), (5, False)])
@pytest.mark.parametrize("what", ["dy", "w", "x"])
@pytest.mark.parametrize("exponent", [-105, -118, -126, -135])
def test_gradients(k, pooled, what, exponent):
    from paper_2409_09083_amd import binding as B
    from paper_2409_09083_amd.harness import Session
    layers = (conv(32, 64, k, slope=1.0),) + ((pool(64),) if pooled else ())
    s = Session(layers, 2, 32, 24, 28, (1, 1), (len(layers),))
    g = torch.Generator().manual_seed(3)
    v = {"x": torch.rand(s.in_shape, generator=g) - 0.5, "w": torch.randn((64, 32, k, k), generator=g) / (6 * k),
         "dy": torch.randn(s.out_shape, generator=g)}
    v[what] = (v[what].double() * 2.0 ** exponent).float()
    s.x.copy_(v["x"])
    s.dy.copy_(v["dy"])
    s.weights = [v["w"].cuda()] + [None] * (len(layers) - 1)
    s.step()
    torch.cuda.synchronize()
    x, w, dz = v["x"].double(), v["w"].double(), v["dy"].double()
    if pooled:
        # (the winners of the pool as the library decided them: products of such small numbers have many equal candidates)
        win = (torch.from_numpy(s.get_boundary(2, B.FTP_BUF_MASK)).long() >> 1) & 3
        full = torch.zeros(dz.shape[0], dz.shape[1], 24, 28, dtype=torch.float64)
        for q in range(4):
            full[:, :, q >> 1::2, q & 1::2] = torch.where(win == q, dz, 0.0)
        dz = full
    got = {"dx": s.dx.cpu().double(), "dw": s.wgrad.cpu().double().reshape(w.shape)}
    s.close()
    ref = {"dx": torch.nn.grad.conv2d_input(x.shape, w, dz, padding=k // 2), "dw": torch.nn.grad.conv2d_weight(x, w.shape, dz, padding=k // 2)}
    for name in ref:
        # ordinary numbers come out within 2e-7 (the norm of the difference over the result's); an entry may be rounded to a multiple of
        # 2^-149 once per partial sum (at most one per 8 products)
        terms = 64 * k * k if name == "dx" else 2 * 24 * 28
        allowed = 1e-6 * float(ref[name].norm()) + (terms / 8) ** 0.5 * 2.0 ** -149 * ref[name].numel() ** 0.5
        assert float((got[name] - ref[name]).norm()) <= allowed, (name, float((got[name] - ref[name]).norm() / ref[name].norm()))
