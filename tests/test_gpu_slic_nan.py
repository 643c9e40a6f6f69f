"""Centres that are NaN of any payload: a pixel takes the first centre in reach when
every distance is NaN, as with the ordinary NaN."""
import numpy as np
import pytest
import torch

from paper_1611_07289_amd import superpixel as sp
from paper_1611_07289_amd import synth

pytestmark = pytest.mark.gpu

BITS = [0x7fc00000, 0xffc00000, 0x7fffffff, 0xffffffff, 0x7fbfffff, 0xffbfffff, 0xfffffffe]


def _nan(bits):
    return np.array([bits], np.uint32).view(np.int32)[0].item()


@pytest.mark.parametrize("h,w,a", [(40, 50, 13), (60, 100, 5)])  # all centres listed; cells near a tile
@pytest.mark.parametrize("column", [2, 3])
def test_centres(h, w, a, column):
    img = torch.from_numpy(synth.slice_images(2, h, w, seed=4)).cuda()
    C = sp.init(img, a, 40.0)
    labels = []
    for bits in BITS:
        Cn = C.clone()
        Cn.view(torch.int32)[..., column] = _nan(bits)
        labels.append(sp.assign(img, Cn, a))
    assert int(labels[0].min()) >= 0
    for bits, lab in zip(BITS, labels):
        assert torch.equal(lab, labels[0]), hex(bits)


@pytest.mark.parametrize("bits", BITS[1:])
def test_images(bits):
    img = torch.from_numpy(synth.slice_images(2, 40, 50, seed=4)).cuda()
    hole = torch.zeros_like(img, dtype=torch.bool)
    hole[:, 5:30, 8:33] = True
    out = []
    for b in (BITS[0], bits):
        I = img.clone()
        I.view(torch.int32)[hole] = _nan(b)
        out.append(sp.slic(I, 13, 40.0, 5.0, iters=3)[0])
    assert torch.equal(out[0], out[1])
