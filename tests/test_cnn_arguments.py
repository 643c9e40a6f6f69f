"""The convolutions take positive sizes only: any other is refused on the host, before
a launch (no GPU is needed for that, and the pointers are never read)."""
import pytest

from paper_1611_07289_amd import pvr

PTR = 1 << 20  # aligned, not memory


@pytest.mark.parametrize("B,H,W", [(0, 8, 8), (4, 0, 8), (4, 8, 0), (4, -1, 8), (4, 8, -7), (-2, 8, 8)])
@pytest.mark.parametrize("cin,cout,s", [(2, 32, 1), (32, 32, 2), (64, 64, 1)])
def test_sizes_that_are_not_positive_are_refused(cin, cout, s, B, H, W):
    L = pvr.load()
    einval = 1
    assert L.pvr_cnn_conv_fwd(PTR, PTR, PTR, PTR, B, H, W, cin, cout, s, 1, None) == einval
    assert L.pvr_cnn_conv_dgrad(PTR, PTR, PTR, PTR, B, H, W, cin, cout, s, None) == einval
    assert L.pvr_cnn_conv_wgrad(PTR, PTR, PTR, PTR, PTR, PTR, B, H, W, cin, cout, s, None) == einval
