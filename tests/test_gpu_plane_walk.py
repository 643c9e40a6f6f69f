"""The plane walk of the Gaussian PSF (2 x 2 samples per lane, one window of
voxels per plane) against the FP64 oracle, where it can go wrong: pixel axes
along the voxel axes in every order and sign (window rows along x and along y,
and patches whose rows run along z, which keep their own walk), odd and tiny
patches, grids smaller than a window, supports reaching outside the grid,
tilts at and beyond the 3- and 4-row windows, other pixel sizes and PSF widths.
FP32 samples to the bar every FP32 simulation is held to (1e-5 of the value,
at least 1e-3 of the largest), the validity exactly, FP64 to 1e-12."""
import numpy as np
import pytest
import torch

import oracle
from paper_1611_07289_amd import pvr, synth
from _gpu import dev, host, sample_close
from test_gpu_gather_blocks import FRAMES, _motion, _problem

pytestmark = pytest.mark.gpu


def _check(g, st, P, theta, f64=True, **plan_args):
    rng = np.random.default_rng(5)
    th = np.asarray(theta, np.float32)
    ctx = oracle.Ctx(g, st, P)
    X = rng.uniform(0.0, 1000.0, (g.nz, g.ny, g.nx)).astype(np.float32)
    ys, Z, val = ctx.simulate(X, th.astype(np.float64))
    plan = pvr.Plan([g], [st], [P], f64=f64)
    plan.build(dev(th))
    y = torch.full((plan.N,), float("nan"), device="cuda")
    e = torch.full_like(y, float("nan"))
    obs = rng.uniform(0.0, 500.0, plan.N).astype(np.float32)
    Xd = dev(X.reshape(-1))
    plan.simulate(Xd, y_obs=dev(obs), y_sim=y, resid=e)
    # a volume of ones simulates to exactly one where valid, to zero elsewhere
    one = torch.empty_like(y)
    plan.simulate(torch.ones_like(Xd), y_sim=one)
    assert np.array_equal(host(one) > 0, val > 0)
    assert np.abs(host(one)[val > 0] - 1).max(initial=0) <= 1e-5
    worst, _ = sample_close(host(y), ys)
    assert worst <= 1e-5
    assert np.array_equal(host(e), np.where(val > 0, obs - host(y), 0).astype(np.float32))
    # the residual statistics the forward pass reduced give the same EM start
    ems = []
    for fresh in (pvr.PVR_EM_RESID_FRESH, 0):
        em = plan.em_state()
        W = torch.empty(plan.M, device="cuda")
        plan.simulate(Xd, y_obs=dev(obs), resid=e)
        plan.robust_weights(e, (yo := dev(obs)), em, None, None, W, pvr.PVR_EM_INIT)
        plan.simulate(Xd, y_obs=yo, resid=e)
        plan.robust_weights(e, yo, em, None, None, W, pvr.PVR_EM_INIT | fresh)
        s = plan.read_em(em)[0]
        ems.append((s.m, s.y_abs_max, s.sigma2))
    assert np.allclose(ems[0], ems[1], rtol=1e-12)
    if f64:
        plan.build(dev(th.astype(np.float64)))
        y64 = torch.full((plan.N,), float("nan"), dtype=torch.float64, device="cuda")
        plan.simulate(dev(X.reshape(-1).astype(np.float64)), y_sim=y64)
        assert np.abs(host(y64) - ys).max() <= 1e-12 * np.abs(ys).max()


@pytest.mark.parametrize("part", range(4))
def test_axes_in_every_order_and_sign(part):
    g, st, P = _problem(FRAMES[part::4], 19, 22, 17)
    _check(g, st, P, _motion(P.M, 10.0, 2.0))


@pytest.mark.parametrize("deg", [0.0, 10.0, 20.0, 30.0, 60.0])
def test_tilts_of_both_windows_and_beyond(deg):
    g, st, P = _problem(synth.orthogonal_frames([30.0, 40.0]), 23, 21, 26)
    _check(g, st, P, _motion(P.M, deg, 3.0))


@pytest.mark.parametrize("spacing,fwhm", [(0.9, (0.9, 1.1, 4.0)), (1.4, (1.4, 1.4, 3.0)),
                                          (1.0, (0.7, 0.7, 2.0)), (1.0, (1.9, 1.9, 4.0)),
                                          (1.0, (1.0, 1.0, 12.0))])
def test_pixels_and_psf_of_other_sizes(spacing, fwhm):
    g, st, P = _problem(synth.orthogonal_frames(), 24, 18, 20, spacing, fwhm)
    _check(g, st, P, _motion(P.M, 8.0, 2.0))


@pytest.mark.parametrize("n", [(8, 8, 8), (3, 9, 40), (2, 2, 2), (64, 5, 16)])
def test_grids_smaller_than_a_window_or_a_support(n):
    g, st, P = _problem(synth.orthogonal_frames(), *n)
    _check(g, st, P, _motion(P.M, 10.0, 2.0))


@pytest.mark.parametrize("w,h", [(16, 16), (17, 16), (32, 31), (33, 33), (64, 64), (63, 5)])
def test_work_items_of_one_to_several_wavefronts(w, h):
    g = synth.iso_grid(72)
    c = synth.grid_center(g)
    st = [synth.make_stack(c, *fr, 64, 64, 3, (1, 1), 4.0, (1.0, 1.0, 4.0))
          for fr in synth.orthogonal_frames()]
    P = synth.Patches(*[np.array(v, np.int32) for v in
                        zip(*[(i, 1, 64 - w, 0, w, h) for i in range(3)])])
    _check(g, st, P, _motion(P.M, 8.0, 2.0), f64=False)


@pytest.mark.parametrize("deg", [0.0, 12.0, 30.0, 60.0])
def test_fp64_motion_derivative_by_finite_differences_of_the_walk(deg):
    # every frame's signs and both windows, patches reaching outside the grid;
    # a central difference of the FP64 simulation is no derivative where a voxel
    # enters or leaves a support, so the loss takes the samples whose value is
    # smooth: those whose differences at two steps agree
    g, st, P = _problem(FRAMES[::5] + synth.orthogonal_frames([35.0]), 21, 18, 24)
    rng = np.random.default_rng(4)
    th = _motion(P.M, deg, 2.0)
    ctx = oracle.Ctx(g, st, P)
    X = rng.uniform(0.0, 1000.0, (g.nz, g.ny, g.nx))
    d = rng.normal(size=(P.M, 6)) * np.array([1e-2] * 3 + [1.0] * 3)  # one direction per patch

    def diff(h):
        yp, _, vp = ctx.simulate(X, th + h * d)
        ym, _, vm = ctx.simulate(X, th - h * d)
        return (yp - ym) / (2 * h), (vp > 0) & (vm > 0)
    d1, v1 = diff(1e-5)
    d2, v2 = diff(2e-6)
    smooth = v1 & v2 & (np.abs(d1 - d2) <= 1e-5 * np.abs(d1).max())
    assert smooth.mean() > 0.5
    gy = np.where(smooth, rng.normal(size=smooth.shape), 0.0)
    plan = pvr.Plan([g], [st], [P], f64=True)
    plan.build(dev(th))
    out = torch.full((P.M, 6), float("nan"), dtype=torch.float64, device="cuda")
    plan.grad_theta(dev(X.reshape(-1)), dev(gy), out)
    off = plan.sample_off
    want = np.array([(gy * d2)[off[s]:off[s + 1]].sum() for s in range(P.M)])
    got = (host(out) * d).sum(1)
    scale = np.array([np.abs(gy * d2)[off[s]:off[s + 1]].sum() for s in range(P.M)])
    assert np.all(np.abs(got - want) <= 1e-5 * np.maximum(scale, 1e-3 * scale.max()))
