"""The scaled copy of dy: every width of a thread's unit, by the planes' pixel count, the storage type and where dy starts, exactly."""
import pytest
import torch

from ftp_synth.configs import conv
from paper_2409_09083_amd import binding as B
from paper_2409_09083_amd.harness import Session

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,h,w,offset,kernel", [
    ("bf16", 12, 20, 0, "k_scale_dy<bf16_t, 8>"), ("bf16", 38, 38, 0, "k_scale_dy<bf16_t, 4>"), ("bf16", 14, 14, 0, "k_scale_dy<bf16_t, 4>"),
    ("bf16", 38, 38, 2, "k_scale_dy<bf16_t, 4>"), ("bf16", 12, 20, 6, "k_scale_dy<bf16_t, 8>"), ("bf16", 38, 38, 1, "k_scale_dy<bf16_t, 1>"),
    ("bf16", 13, 15, 0, "k_scale_dy<bf16_t, 1>"), ("f32", 14, 14, 0, "k_scale_dy<float, 4>"), ("f32", 14, 14, 1, "k_scale_dy<float, 4>"), ("f32", 13, 14, 0, "k_scale_dy<float, 1>")])
@pytest.mark.parametrize("cout", [16, 37])
def test_scaled_copy(dtype, h, w, offset, kernel, cout):
    """offset: elements between a 16-byte boundary and dy."""
    g = torch.Generator(device="cuda").manual_seed(6)
    s = Session((conv(16, cout, 1, slope=0.3),), 3, 16, h, w, (1, 2), (1,), dtype)
    s.x.normal_(generator=g)
    s.weights = [(torch.randn((cout, 16, 1, 1), device="cuda", generator=g) / 4).to(s.tdtype)]
    n = s.dy.numel()
    s.dy = torch.empty(n + 8, dtype=s.tdtype, device="cuda")[offset:offset + n].view(s.out_shape)
    s.dy.normal_(generator=g)
    s.forward()
    B.ftp_profile(s.plan, 1)
    s.backward()
    torch.cuda.synchronize()
    assert [r["kernel"] for r in B.ftp_profile_read(s.plan) if r["pass"] == "scale_dy"] == [kernel]
    scaled = s._buffer(1, B.FTP_BUF_DELTA)[0]
    # (products in fp32, rounded once to the storage type)
    assert torch.equal(scaled.view(s.out_shape), torch.where(s.y > 0, s.dy, (s.dy.float() * torch.tensor(0.3, device="cuda")).to(s.tdtype)))
    s.close()


@pytest.mark.parametrize("dtype,h,w,offset,cout,kernel", [
    # 128 MB and just below, units of 16 and of 8 bytes, dy on a dword that is no quad; then a map of a tenth of that
    ("bf16", 600, 556, 0, 64, "k_scale_dy<bf16_t, 8, past>"), ("bf16", 600, 555, 2, 64, "k_scale_dy<bf16_t, 8>"), ("bf16", 806, 806, 2, 33, "k_scale_dy<bf16_t, 4, past>"),
    ("f32", 600, 556, 1, 32, "k_scale_dy<float, 4, past>"), ("f32", 600, 555, 0, 32, "k_scale_dy<float, 4>"), ("f32", 152, 152, 0, 64, "k_scale_dy<float, 4>")])
def test_scaled_copy_of_large_maps(dtype, h, w, offset, cout, kernel):
    """Maps that the caches cannot hold beside their copy are read past them, others through them."""
    test_scaled_copy(dtype, h, w, offset, kernel, cout)
