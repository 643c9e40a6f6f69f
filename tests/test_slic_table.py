"""The pack table of superpixel boxes, written by 8-byte columns, against the same
table by stacked columns: element types, layouts and orders of the boxes, empty
superpixels, no superpixel at all."""
import numpy as np
import pytest

from paper_1611_07289_amd.superpixel import patch_table


def _boxes(n, *shape):
    return np.random.default_rng(n).integers(-3, 200, (n, *shape, 4))


@pytest.mark.parametrize("B", [
    _boxes(5, 7).astype(np.int32), np.abs(_boxes(5, 7)).astype(np.int32) + 1, _boxes(1, 300),
    _boxes(4, 3, 5).astype(np.int16), _boxes(6, 9).astype(np.float32) + 0.5,
    np.asfortranarray(_boxes(6, 9).astype(np.int32)), _boxes(8, 10).astype(np.int32)[::-2, 1::3],
    _boxes(6, 9).astype(">i4"), np.zeros((3, 4, 4), np.int32), np.zeros((3, 0, 4), np.int32)])
def test_table_equals_stacked_columns(B):
    flat = B.reshape(B.shape[0], B.size // (4 * B.shape[0]), 4)
    im, k = np.nonzero(flat[:, :, 2] > 0)
    want = np.column_stack([im, k, flat[im, k]]).astype(np.int32)
    got = patch_table(B) if B.size else patch_table(flat)
    assert got.dtype == np.int32 and got.shape == want.shape and got.flags.c_contiguous
    assert np.array_equal(got, want)
