"""The tiled convolutions (forward, data and weight gradient) where their tiles
end: images of one pixel, within, at and past the 8 x 8 and 16 x 16 tiles,
odd sides, one to many images.  Against FP64 on the same BF16 operands: every
output within the rounding bound of its own FP32 sum ((n + 2) 2^-24 of the sum
of magnitudes of its n terms) and, where it is stored in BF16, half a unit in
the last place (2^-8 of the value, which also covers the smallest normals).
The first two layers in one pass are the two layers bit for bit."""
import pytest
import torch
import torch.nn.functional as F

from paper_1611_07289_amd import pvr

pytestmark = pytest.mark.gpu

SHAPES = [(2, 32, 1), (32, 32, 2), (32, 64, 1), (64, 64, 2), (64, 64, 1), (32, 32, 1), (64, 32, 1)]
SIZES = [(1, 1, 1), (5, 8, 8), (3, 5, 7), (9, 9, 8), (2, 16, 16), (3, 17, 15), (1, 33, 18),
         (2, 15, 35), (70, 8, 7), (66, 16, 3), (257, 7, 8), (258, 16, 15)]


def _st():
    return torch.cuda.current_stream().cuda_stream


def _data(cin, cout, s, B, H, W):
    g = torch.Generator().manual_seed(B * 1000 + H * 10 + W + cin + cout + s)
    Ho, Wo = (H - 1) // s + 1, (W - 1) // s + 1
    x = torch.randn(B, H, W, cin, generator=g).bfloat16()
    w = (torch.randn(cout, 3, 3, cin, generator=g) * 0.1).bfloat16()
    b = torch.randn(cout, generator=g) * 0.1
    o = torch.randn(B, Ho, Wo, cout, generator=g).bfloat16()
    go = torch.randn(B, Ho, Wo, cout, generator=g).bfloat16()
    return x, w, b, o, go


def _nchw(t):
    return t.double().permute(0, 3, 1, 2)


def _ok(got, ref, mag, n, stored):
    got, ref, mag = got.double().cpu(), ref.double(), mag.double()
    bar = (n + 2) * 2.0 ** -24 * mag + (2.0 ** -8 if stored else 2.0 ** -23) * ref.abs() + 1e-37
    assert bool(torch.all((got - ref).abs() <= bar)), float(((got - ref).abs() / bar).max())


@pytest.mark.parametrize("cin,cout,s", SHAPES)
@pytest.mark.parametrize("B,H,W", SIZES)
def test_forward(cin, cout, s, B, H, W):
    x, w, b, o, _ = _data(cin, cout, s, B, H, W)
    out = torch.full_like(o, float("nan")).cuda()
    xd, wd, bd = x.cuda(), w.cuda(), b.cuda()
    for relu in (0, 1):
        pvr._check(pvr.load().pvr_cnn_conv_fwd(xd.data_ptr(), wd.data_ptr(), bd.data_ptr(),
                                               out.data_ptr(), B, H, W, cin, cout, s, relu, _st()))
        ref = F.conv2d(_nchw(x), _nchw(w), b.double(), stride=s, padding=1)
        mag = F.conv2d(_nchw(x).abs(), _nchw(w).abs(), b.double().abs(), stride=s, padding=1)
        if relu:
            ref = ref.clamp_min(0)
        _ok(out, ref.permute(0, 2, 3, 1), mag.permute(0, 2, 3, 1), 9 * cin + 1, True)


@pytest.mark.parametrize("cin,cout,s", SHAPES)
@pytest.mark.parametrize("B,H,W", SIZES)
def test_gradients(cin, cout, s, B, H, W):
    x, w, b, o, go = _data(cin, cout, s, B, H, W)
    L = pvr.load()
    gp = _nchw(go) * (_nchw(o) > 0)
    xd, od, gd = x.cuda(), o.cuda(), go.cuda()
    if cin >= 16:
        wt = w.permute(1, 2, 3, 0).contiguous().cuda()
        gin = torch.full_like(x, float("nan")).cuda()
        pvr._check(L.pvr_cnn_conv_dgrad(gd.data_ptr(), od.data_ptr(), wt.data_ptr(), gin.data_ptr(),
                                        B, H, W, cin, cout, s, _st()))
        op = ((H - 1) % s, (W - 1) % s)
        ref = F.conv_transpose2d(gp, _nchw(w), stride=s, padding=1, output_padding=op)
        mag = F.conv_transpose2d(gp.abs(), _nchw(w).abs(), stride=s, padding=1, output_padding=op)
        _ok(gin, ref.permute(0, 2, 3, 1), mag.permute(0, 2, 3, 1), 9 * cout, True)
    scr = torch.full((L.pvr_cnn_wgrad_scratch(B, H, W, cin, cout, s) // 4 + 4,), float("nan"),
                     device="cuda")
    dw, db = torch.full((cout, 3, 3, cin), float("nan"), device="cuda"), torch.empty(cout, device="cuda")
    pvr._check(L.pvr_cnn_conv_wgrad(gd.data_ptr(), od.data_ptr(), xd.data_ptr(), scr.data_ptr(),
                                    dw.data_ptr(), db.data_ptr(), B, H, W, cin, cout, s, _st()))

    def wgrad(a, g):
        return torch.nn.grad.conv2d_weight(a, (cout, cin, 3, 3), g, stride=s, padding=1).permute(0, 2, 3, 1)

    n = gp.shape[0] * gp.shape[2] * gp.shape[3]
    _ok(dw, wgrad(_nchw(x), gp), wgrad(_nchw(x).abs(), gp.abs()), n, False)
    _ok(db, gp.sum((0, 2, 3)), gp.abs().sum((0, 2, 3)), n, False)


@pytest.mark.parametrize("B,H,W", SIZES + [(1, 64, 64), (3, 63, 34), (200, 16, 34)])
def test_first_two_layers_in_one_pass(B, H, W):
    L = pvr.load()
    x, w1, b1, o1, _ = _data(2, 32, 1, B, H, W)
    _, w2, b2, o2, _ = _data(32, 32, 2, B, H, W)
    xd, w1, b1, w2, b2 = (t.cuda() for t in (x, w1, b1, w2, b2))
    mid, two, one = o1.cuda(), torch.empty_like(o2, device="cuda"), torch.empty_like(o2, device="cuda")
    pvr._check(L.pvr_cnn_conv_fwd(xd.data_ptr(), w1.data_ptr(), b1.data_ptr(), mid.data_ptr(), B, H,
                                  W, 2, 32, 1, 1, _st()))
    pvr._check(L.pvr_cnn_conv_fwd(mid.data_ptr(), w2.data_ptr(), b2.data_ptr(), two.data_ptr(), B, H,
                                  W, 32, 32, 2, 1, _st()))
    pvr._check(L.pvr_cnn_stem_fwd(xd.data_ptr(), w1.data_ptr(), b1.data_ptr(), w2.data_ptr(),
                                  b2.data_ptr(), one.data_ptr(), B, H, W, _st()))
    assert torch.equal(two, one)
