"""The SLIC kernels where their paths change: batches of fewer and more images
than are shared out to the chip's eight L2 caches (every image as it comes out
alone, bit for bit), more centres than are listed at once, windows beyond the
32-bit sums, NaN pixels; and the packing at the edges of its 64-pixel words,
row groups, quads and dilation limit (integer and copy work: bit-exact against
a separable dilation), with more patches than one round of the offsets."""
import numpy as np
import pytest
import torch
from scipy import ndimage

from oracle import slic as oslic
from paper_1611_07289_amd import superpixel as sp
from paper_1611_07289_amd import synth
from test_gpu_slic import _check_assignment

pytestmark = pytest.mark.gpu

T0, TMIN = 40.0, 5.0


@pytest.mark.parametrize("n", [7, 8, 9, 17])
@pytest.mark.parametrize("h,w,a", [(33, 70, 9), (64, 96, 5), (40, 31, 17)])  # 32, 260 and 6 centres
def test_every_image_of_a_batch_as_alone(n, h, w, a):
    I = torch.from_numpy(synth.slice_images(n, h, w, seed=3)).cuda()
    lab, C = sp.slic(I, a, T0, TMIN, iters=3)
    B = sp.boxes(lab, C, a, 2)
    for i in range(n):
        l1, c1 = sp.slic(I[i:i + 1], a, T0, TMIN, iters=3)
        assert torch.equal(lab[i:i + 1], l1) and torch.equal(C[i:i + 1], c1)
        assert torch.equal(B[i:i + 1], sp.boxes(l1, c1, a, 2))
    img = I[0].double().cpu().numpy()
    _check_assignment(img, C[0].double().cpu().numpy(), lab[0].cpu().numpy(), a)


@pytest.mark.parametrize("h,w,a", [(30, 1100, 512), (30, 1100, 513), (1100, 30, 600)])
def test_windows_around_the_32_bit_sums(h, w, a):
    I = synth.slice_images(2, h, w, seed=9)
    Ig = torch.from_numpy(I).cuda()
    C0 = sp.init(Ig, a, T0)
    lab = sp.assign(Ig, C0, a)
    C1 = sp.update(Ig, lab, C0.clone(), a, TMIN).cpu().numpy()
    for i in range(2):
        ref = oslic.update(I[i].astype(np.float64), lab[i].cpu().numpy(),
                           C0[i].cpu().numpy().astype(np.float64), TMIN)
        # FP64 sums, stored in FP32: half a unit in the last place
        assert np.all(np.abs(C1[i] - ref) <= 2.0 ** -23 * np.abs(ref))


def test_nan_pixels_join_the_first_centre_that_covers_them():
    I = synth.slice_images(1, 48, 48, seed=4)
    C = sp.init(torch.from_numpy(I).cuda(), 12, T0)
    I[0, 20, 13] = np.nan
    lab = sp.assign(torch.from_numpy(I).cuda(), C, 12).cpu().numpy()[0]
    c = C[0].cpu().numpy()
    cover = np.nonzero((np.abs(13 - c[:, 0]) <= 12) & (np.abs(20 - c[:, 1]) <= 12))[0]
    assert lab[20, 13] == cover[0]
    I[0, 20, 13] = 0.0
    ref = sp.assign(torch.from_numpy(I).cuda(), C, 12).cpu().numpy()[0]
    ref[20, 13] = cover[0]
    assert np.array_equal(lab, ref)


def _pack_check(I, lab, gamma, tab):
    y, m = sp.pack(torch.from_numpy(I).cuda(), torch.from_numpy(lab).cuda(), gamma, tab)
    y, m = y.cpu().numpy(), m.cpu().numpy()
    o = 0
    for im, k, x0, y0, w, h in tab:
        box = (im, slice(y0, y0 + h), slice(x0, x0 + w))
        want = (lab[box] == k).astype(np.uint8)
        want = ndimage.maximum_filter1d(want, 2 * gamma + 1, axis=0, mode="constant")
        want = ndimage.maximum_filter1d(want, 2 * gamma + 1, axis=1, mode="constant")
        assert np.array_equal(m[o:o + w * h].reshape(h, w), want), (gamma, w, h)
        assert np.array_equal(y[o:o + w * h].reshape(h, w), I[box]), (gamma, w, h)
        o += w * h
    assert o == y.size == m.size


@pytest.mark.parametrize("gamma", [0, 1, 3, 4, 19, 38, 63, 64, 90])
def test_pack_at_the_edges_of_words_rows_and_quads(gamma):
    rng = np.random.default_rng(gamma)
    I = rng.normal(size=(3, 150, 210)).astype(np.float32)
    lab = np.full((3, 150, 210), -1, np.int32)
    lab[rng.random(lab.shape) < 2e-3] = 0
    lab[rng.random(lab.shape) < 2e-3] = 1
    rows = []
    for w in (1, 2, 3, 4, 5, 63, 64, 65, 127, 128, 129, 193):
        for h in (1, 2, 7, 8, 9, 31, 32, 33, 130):
            x0, y0 = rng.integers(0, 210 - w + 1), rng.integers(0, 150 - h + 1)
            rows.append((len(rows) % 3, len(rows) % 2, x0, y0, w, h))
    _pack_check(I, lab, gamma, np.array(rows, np.int32))


def test_pack_a_box_of_more_words_than_the_bit_rows_hold():
    rng = np.random.default_rng(2)
    I = rng.normal(size=(1, 2100, 3)).astype(np.float32)
    lab = (rng.random((1, 2100, 3)) < 5e-3).astype(np.int32)
    for h in (2048, 2049):
        _pack_check(I, lab, 5, np.array([(0, 1, 1, 7, 2, h), (0, 1, 0, 3, 3, 100)], np.int32))


def test_pack_offsets_of_many_patches():
    rng = np.random.default_rng(6)
    M = 2 * 16384 + 77
    I = rng.normal(size=(1, 64, 64)).astype(np.float32)
    lab = rng.integers(0, 2, (1, 64, 64)).astype(np.int32)
    w, h = rng.integers(1, 6, M), rng.integers(1, 4, M)
    tab = np.column_stack([np.zeros(M), rng.integers(0, 2, M), rng.integers(0, 59, M),
                           rng.integers(0, 60, M), w, h]).astype(np.int32)
    y, m = sp.pack(torch.from_numpy(I).cuda(), torch.from_numpy(lab).cuda(), 0, tab)
    q = np.arange(w.astype(np.int64) @ h)
    off = np.concatenate([[0], np.cumsum(w.astype(np.int64) * h)])
    s = np.searchsorted(off, q, side="right") - 1
    r, c = np.divmod(q - off[s], w[s])
    yy, xx = tab[s, 3] + r, tab[s, 2] + c
    assert np.array_equal(y.cpu().numpy(), I[0, yy, xx])
    assert np.array_equal(m.cpu().numpy(), (lab[0, yy, xx] == tab[s, 1]).astype(np.uint8))
