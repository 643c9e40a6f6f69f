"""Patches whose motion takes them off the shared windows (the plane walk and the
block gather), which the same kernels then take sample by sample and voxel by
voxel: work items of one to several wavefronts, odd sides and a second item, and
stacks whose patches are on and off the windows in turn, so that a lane's sums
change hands between them.  The bars are those of the two kernels' own tests."""
import numpy as np
import pytest

from paper_1611_07289_amd import synth
from test_gpu_gather_blocks import _check as check_gather
from test_gpu_gather_blocks import _motion, _problem
from test_gpu_plane_walk import _check as check_forward

pytestmark = pytest.mark.gpu


def _patches(w, h):
    g = synth.iso_grid(72)
    c = synth.grid_center(g)
    st = [synth.make_stack(c, *fr, 64, 64, 3, (1, 1), 4.0, (1.0, 1.0, 4.0))
          for fr in synth.orthogonal_frames()]
    P = synth.Patches(*[np.array(v, np.int32) for v in
                        zip(*[(i, 1, 64 - w, 0, w, h) for i in range(3)])])
    return g, st, P


@pytest.mark.parametrize("w,h", [(16, 16), (17, 16), (32, 31), (33, 33), (64, 64), (63, 5)])
def test_work_items_off_the_walk(w, h):
    g, st, P = _patches(w, h)
    th = _motion(P.M, 1.0, 2.0)
    th[:, 0] += np.radians(40.0)
    th[:, 1] += np.radians(-35.0)
    check_forward(g, st, P, th)
    check_gather(g, st, P, th)


@pytest.mark.parametrize("sinc", [False, True])
def test_patches_on_and_off_the_windows_in_turn(sinc):
    g, st, P = _problem(synth.orthogonal_frames([30.0]), 23, 21, 26)
    rep = 3
    P = synth.Patches(*[np.repeat(np.asarray(a), rep) for a in (P.stack, P.slice, P.x0, P.y0, P.w, P.h)])
    th = _motion(P.M, 6.0, 3.0)
    far = _motion(P.M, 70.0, 3.0, seed=8)
    th[1::2] = far[1::2]
    check_gather(g, st, P, th, sinc=sinc, f64=not sinc)
    if not sinc:
        check_forward(g, st, P, th)
