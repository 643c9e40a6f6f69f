"""How many pixels a weight's gradient adds up in FP32 before its sum goes on in
FP64: at most as many as 256 KS blocks of a layer hold (KS sets of wavefronts, of 32
pixels a step).  Operands are whole numbers whose sum over that many pixels stays
below 2^24, so that such a sum is exact and the gradient is the exact sum, rounded
once; over twice as many it passes 2^24 and loses its odd part."""
import pytest
import torch
import torch.nn.functional as F

from paper_1611_07289_amd import pvr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin,cout,s,B,H,W", [
    (64, 64, 1, 256, 16, 16), (64, 64, 1, 1024, 8, 8), (64, 64, 1, 300, 13, 15), (64, 64, 2, 256, 16, 16),
    (32, 64, 1, 256, 16, 16), (64, 32, 1, 256, 16, 16), (32, 32, 2, 256, 32, 32), (32, 32, 1, 256, 32, 32),
    (32, 32, 1, 1100, 8, 7), (64, 64, 1, 3, 100, 90), (32, 64, 1, 1, 5, 5), (2, 32, 1, 256, 16, 16)])
def test_a_gradient_of_whole_numbers_is_exact(cin, cout, s, B, H, W):
    Ho, Wo = (H - 1) // s + 1, (W - 1) // s + 1
    P, ks = B * Ho * Wo, 16 if cin < 32 else 16 // (cin // 16 * cout // 16)
    step = 32 * ks
    chain = max(step, ((P + 255) // 256 + step - 1) // step * step) // ks
    top = min(255, int((2 ** 24 / chain) ** 0.5))
    gen = torch.Generator().manual_seed(P + cin)
    x = torch.randint(top - top // 4, top + 1, (B, H, W, cin), generator=gen).bfloat16()
    g = torch.randint(top - top // 4, top + 1, (B, Ho, Wo, cout), generator=gen).bfloat16()
    assert chain * top * top < 2 ** 24 and float(x.max()) <= top and float(g.max()) <= top
    xd, gd, od = x.cuda(), g.cuda(), torch.ones_like(g).cuda()
    L = pvr.load()
    scr = torch.full((L.pvr_cnn_wgrad_scratch(B, H, W, cin, cout, s) // 4 + 4,), float("nan"), device="cuda")
    dw = torch.full((cout, 3, 3, cin), float("nan"), device="cuda")
    db = torch.full((cout,), float("nan"), device="cuda")
    pvr._check(L.pvr_cnn_conv_wgrad(gd.data_ptr(), od.data_ptr(), xd.data_ptr(), scr.data_ptr(),
                                    dw.data_ptr(), db.data_ptr(), B, H, W, cin, cout, s,
                                    torch.cuda.current_stream().cuda_stream))
    xp = F.pad(x.double(), (0, 0, 1, 1, 1, 1))
    go = g.double().reshape(-1, cout)
    ref = torch.stack([go.t() @ xp[:, ky:ky + s * (Ho - 1) + 1:s, kx:kx + s * (Wo - 1) + 1:s].reshape(-1, cin)
                       for ky in range(3) for kx in range(3)], 1).reshape(cout, 3, 3, cin)
    assert torch.equal(dw.cpu(), ref.float())
    assert torch.equal(db.cpu(), go.sum(0).float())
