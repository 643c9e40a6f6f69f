"""The block gather of the adjoint (2 x 2 voxels per lane, one pixel window for
the four) against the FP64 oracle, where it can go wrong: stacks whose pixel
axes run along the voxel axes in every order and sign, ragged grids (partial
bricks) and patches (1 x 1, strips, odd sides, reaching outside the grid),
tilts beyond the shared window (the per-voxel walk inside the kernel), a mix
of both in one plan, and pixels of another size than the voxels (the
per-voxel kernel).  FP32 voxels to the adjoint bar of _tolerance.py (the
rounding bound every FP32 gather is held to), FP64 to 1e-12 of the scale
(A^T |r|) it bounds."""
import itertools

import numpy as np
import pytest
import torch

import oracle
from paper_1611_07289_amd import pvr, synth
from _gpu import dev, host
from _tolerance import adjoint_bar

pytestmark = pytest.mark.gpu

E = np.eye(3)
# every signed permutation of the voxel axes with n = +-(e1 x e2)
FRAMES = [(s0 * E[p[0]], s1 * E[p[1]], s2 * E[p[2]])
          for p in itertools.permutations(range(3))
          for s0, s1, s2 in [(1, 1, 1), (-1, 1, 1), (1, -1, -1), (-1, -1, 1)]]


def _problem(frames, nx, ny, nz, spacing=1.0, fwhm=(1.0, 1.0, 4.0)):
    v2w = np.zeros((3, 4))
    v2w[0, 0] = v2w[1, 1] = v2w[2, 2] = 1.0
    g = synth.Grid(nx, ny, nz, v2w)
    c = synth.grid_center(g)
    st = [synth.make_stack(c, *fr, 21, 17, 5, (spacing, spacing), 4.0, fwhm) for fr in frames]
    rows = []
    for i in range(len(st)):
        rows += [(i, 2, 3, 2, 13, 11), (i, 1, 0, 0, 21, 17), (i, 3, 5, 6, 1, 1), (i, 2, 0, 7, 21, 1),
                 (i, 0, 9, 0, 1, 17), (i, 4, 15, 11, 6, 6)]
    return g, st, synth.Patches(*[np.array(v, np.int32) for v in zip(*rows)])


def _check(g, st, P, theta, sinc=False, f64=True, blocks=None):
    rng = np.random.default_rng(11)
    th = np.asarray(theta, np.float32)
    ctx = oracle.Ctx(g, st, P, psf="sinc") if sinc else oracle.Ctx(g, st, P)
    plan = pvr.Plan([g], [st], [P], f64=f64)
    if sinc:
        plan.set_psf(pvr.PVR_PSF_SINC)
    r = rng.normal(size=plan.N).astype(np.float32)
    q = rng.uniform(0.1, 1.0, plan.N).astype(np.float32)
    W = rng.uniform(0.2, 1.0, plan.M).astype(np.float32)
    W[1] = 0.0
    n_off = plan.sample_off
    Wj = np.repeat(W, np.diff(n_off))
    wn, wd = (W64 := Wj.astype(np.float64)) * q * r, W64 * q
    on = ctx.backproject(th.astype(np.float64), wn).reshape(-1)
    od = ctx.backproject(th.astype(np.float64), wd).reshape(-1)
    plan.build(dev(th))
    num, den, only = (torch.full((plan.V,), float("nan"), device="cuda") for _ in range(3))
    plan.backproject(dev(r), dev(q), dev(W), num, den)
    plan.backproject(dev(r), dev(q), dev(W), only, None)
    bar = adjoint_bar(ctx, th.astype(np.float64), wn)
    bad = adjoint_bar(ctx, th.astype(np.float64), wd)
    floor = 1e-12 * max(float(np.abs(on).max()), 1e-30)
    assert np.all(np.abs(host(num) - on) <= bar + floor)
    assert np.all(np.abs(host(den) - od) <= bad + floor)
    assert torch.equal(num, only)  # the denominator does not change the numerator
    if f64:
        plan.build(dev(th.astype(np.float64)))
        n64, d64 = (torch.full((plan.V,), float("nan"), dtype=torch.float64, device="cuda")
                    for _ in range(2))
        plan.backproject(dev(r.astype(np.float64)), dev(q.astype(np.float64)),
                         dev(W.astype(np.float64)), n64, d64)
        scale = ctx.backproject(th.astype(np.float64), np.abs(wn)).max()
        assert np.abs(host(n64) - on).max() <= 1e-12 * scale
        assert np.abs(host(d64) - od).max() <= 1e-12 * np.abs(od).max()


def _motion(M, deg, mm, seed=3):
    return synth.random_motion_batch(M, deg, mm, seed)


@pytest.mark.parametrize("part", range(4))
def test_axes_in_every_order_and_sign(part):
    g, st, P = _problem(FRAMES[part::4], 19, 22, 17)
    _check(g, st, P, _motion(P.M, 10.0, 2.0))


@pytest.mark.parametrize("sinc", [False, True])
@pytest.mark.parametrize("deg", [0.0, 10.0, 25.0, 60.0])
def test_tilts_inside_and_beyond_the_shared_window(deg, sinc):
    frames = synth.orthogonal_frames([30.0])
    g, st, P = _problem(frames, 23, 21, 26)
    _check(g, st, P, _motion(P.M, deg, 3.0), sinc=sinc, f64=not sinc)


@pytest.mark.parametrize("spacing,fwhm", [(0.9, (0.9, 1.1, 4.0)), (1.4, (1.4, 1.4, 3.0)),
                                          (1.0, (0.7, 0.7, 2.0)), (1.0, (1.9, 1.9, 4.0))])
def test_pixels_and_psf_of_other_sizes(spacing, fwhm):
    g, st, P = _problem(synth.orthogonal_frames(), 24, 18, 20, spacing, fwhm)
    _check(g, st, P, _motion(P.M, 8.0, 2.0))


@pytest.mark.parametrize("n", [(8, 8, 8), (1, 9, 40), (64, 8, 16)])
def test_grids_of_few_and_partial_bricks(n):
    g, st, P = _problem(synth.orthogonal_frames(), *n)
    _check(g, st, P, _motion(P.M, 10.0, 2.0), f64=False)


def test_a_non_finite_input_stays_where_its_support_is():
    # one patch; a NaN sample reaches only voxels of its own layer range
    g, st, _ = _problem(synth.orthogonal_frames()[:1], 24, 24, 24)
    P = synth.Patches(*[np.array([v], np.int32) for v in (0, 2, 2, 2, 15, 13)])
    plan = pvr.Plan([g], [st], [P])
    plan.build(torch.zeros(1, 6, device="cuda"))
    e = torch.ones(plan.N, device="cuda")
    e[6 * 15 + 7] = float("nan")
    num = torch.empty(plan.V, device="cuda")
    plan.backproject(e, None, None, num, None)
    bad = torch.isnan(num).reshape(24, 24, 24).nonzero().cpu().numpy()
    # slice 2 of 5 at 4 mm lies at z = 11.5; 3 sigma through-plane is 5.1 mm
    assert bad.size and np.all(np.abs(bad[:, 0] - 11.5) <= 5.1)
    assert len(np.unique(bad[:, 1])) <= 4 and len(np.unique(bad[:, 2])) <= 4


@pytest.mark.parametrize("spacing", [1.0, 1.8])  # halves of the block gather, sub-bricks of the other
@pytest.mark.parametrize("n", [63, 64, 65, 700])
def test_lists_up_to_more_patches_than_a_brick_holds_in_lds(n, spacing):
    # n patches over every brick (more than 512 hits test their patches again)
    g, st, P = _problem(synth.orthogonal_frames()[:1], 9, 8, 8, spacing, (spacing, spacing, 4.0))
    P = synth.Patches(*[np.resize(np.asarray(a)[:2], n) for a in
                        (P.stack, P.slice, P.x0, P.y0, P.w, P.h)])
    th = _motion(n, 6.0, 1.0)
    _check(g, st, P, th, f64=False)
    plan = pvr.Plan([g], [st], [P])
    r = dev(np.random.default_rng(5).normal(size=plan.N).astype(np.float32))
    out = []
    for _ in range(3):  # the lists are made anew: the same lists, the same sums
        plan.build(dev(np.asarray(th, np.float32)))
        out.append(torch.empty(plan.V, device="cuda"))
        plan.backproject(r, None, None, out[-1], None)
    assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])
