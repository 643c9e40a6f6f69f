"""The block gather with a brick's lists split over 8, 4, 2 and 1 parts: thin ragged
grids just below and at the brick numbers where the split changes (256, 4096 and 8192;
FP64 has four parts at most), against the FP64 oracle to the bars of the gather: axes of
several orders and signs, tilts within and beyond the shared window in one plan, partial
bricks."""
import pytest

from test_gpu_gather_blocks import FRAMES, _check, _motion, _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("by,bz", [(15, 17), (16, 16), (63, 65), (64, 64), (63, 130), (64, 128)])
def test_every_split_of_the_lists(by, bz):
    g, st, P = _problem(FRAMES[1::5], 3, 8 * by - 3, 8 * bz - 7)
    th = _motion(P.M, 10.0, 2.0)
    th[::3] = _motion(P.M, 50.0, 2.0, 9)[::3]
    _check(g, st, P, th)
