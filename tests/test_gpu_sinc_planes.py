"""The sinc PSF's walk by planes against the FP64 oracle, where it can go wrong:
pixel axes along the voxel axes in every order and sign (both volume copies, and
patches whose rows run along z, which keep the row walk), tilts at and beyond its
reach, pixels and zeros of other sizes, supports reaching outside the grid, grids
smaller than a support.  FP32 samples to the bar every FP32 simulation is held to
(1e-5 of the value, at least 1e-3 of the largest), the validity exactly, the
adjoint of the same plan by the bar of tests/_tolerance.py."""
import numpy as np
import pytest
import torch

import oracle
from paper_1611_07289_amd import pvr, synth
from _gpu import dev, host, sample_close
from _tolerance import adjoint_bar
from test_gpu_gather_blocks import FRAMES, _motion, _problem

pytestmark = pytest.mark.gpu


def _check(g, st, P, theta):
    rng = np.random.default_rng(6)
    th = np.asarray(theta, np.float32)
    t64 = th.astype(np.float64)
    ctx = oracle.Ctx(g, st, P, psf="sinc")
    X = rng.uniform(0.0, 1000.0, (g.nz, g.ny, g.nx)).astype(np.float32)
    ys, Z, val = ctx.simulate(X, t64)
    plan = pvr.Plan([g], [st], [P])
    plan.set_psf(pvr.PVR_PSF_SINC)
    plan.build(dev(th))
    y = torch.full((plan.N,), float("nan"), device="cuda")
    Xd = dev(X.reshape(-1))
    plan.simulate(Xd, y_sim=y)
    one = torch.empty_like(y)
    plan.simulate(torch.ones_like(Xd), y_sim=one)
    assert np.array_equal(host(one) > 0, val > 0)
    assert np.abs(host(one)[val > 0] - 1).max(initial=0) <= 1e-5
    worst, _ = sample_close(host(y), ys)
    assert worst <= 1e-5
    r = rng.normal(size=plan.N)
    num = torch.empty(plan.V, device="cuda")
    plan.backproject(dev(r.astype(np.float32)), num=num)
    r = r.astype(np.float32).astype(np.float64)
    want = ctx.backproject(t64, r).reshape(-1)
    assert float((np.abs(host(num) - want) / (adjoint_bar(ctx, t64, r) + 1e-30)).max()) <= 1.0


@pytest.mark.parametrize("part", range(4))
def test_axes_in_every_order_and_sign(part):
    g, st, P = _problem(FRAMES[part::4], 19, 22, 17)
    _check(g, st, P, _motion(P.M, 10.0, 2.0))


@pytest.mark.parametrize("deg", [0.0, 10.0, 20.0, 30.0, 60.0])
def test_tilts_within_reach_and_beyond(deg):
    g, st, P = _problem(synth.orthogonal_frames([30.0, 40.0]), 23, 21, 26)
    _check(g, st, P, _motion(P.M, deg, 3.0))


@pytest.mark.parametrize("spacing,fwhm", [(0.9, (0.9, 1.1, 4.0)), (1.4, (1.4, 1.4, 3.0)),
                                          (1.0, (0.7, 0.7, 2.0)), (1.0, (1.3, 1.3, 4.0)),
                                          (1.0, (1.9, 1.9, 4.0)), (1.0, (1.0, 1.0, 0.8)),
                                          (1.0, (1.0, 1.0, 12.0))])
def test_pixels_and_psf_of_other_sizes(spacing, fwhm):
    g, st, P = _problem(synth.orthogonal_frames(), 24, 18, 20, spacing, fwhm)
    _check(g, st, P, _motion(P.M, 8.0, 2.0))


@pytest.mark.parametrize("n", [(8, 8, 8), (3, 9, 40), (2, 2, 2), (64, 5, 16)])
def test_grids_smaller_than_a_support(n):
    g, st, P = _problem(synth.orthogonal_frames(), *n)
    _check(g, st, P, _motion(P.M, 10.0, 2.0))
