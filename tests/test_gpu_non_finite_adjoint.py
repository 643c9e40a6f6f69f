"""How far a sample that is not finite reaches in the adjoint.  The block gather
weighs whole windows, by zero outside a support, and zero times NaN is NaN: what is
poisoned has to be no more than the gather of a single voxel poisons, the voxels
whose nearest pixel lies within one of the sample's in u and v (FP64, whose inputs
are packed without padding: within one of it in the packed order, across patches)
and whose distance from its plane is within the support."""
import numpy as np
import pytest
import torch

import oracle
from paper_1611_07289_amd import pvr, synth
from _gpu import dev, host
from test_gpu_gather_blocks import _motion, _problem
from test_gpu_non_finite import K, _rotation

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("sinc", [False, True])
def test_adjoint(sinc, f64):
    g, st, P = _problem(synth.orthogonal_frames([30.0]), 24, 22, 26)
    th = _motion(P.M, 9.0, 1.5).astype(np.float32).astype(np.float64)
    ctx = oracle.Ctx(g, st, P, psf="sinc") if sinc else oracle.Ctx(g, st, P)
    plan = pvr.Plan([g], [st], [P], f64=f64)
    if sinc:
        plan.set_psf(pvr.PVR_PSF_SINC)
    plan.build(dev(th if f64 else th.astype(np.float32)))
    dt = torch.float64 if f64 else torch.float32
    rng = np.random.default_rng(9)
    e = rng.normal(size=plan.N)
    val = ctx.simulate(np.ones((g.nz, g.ny, g.nx), np.float32), th)[2] > 0
    z, y, x = np.meshgrid(*(np.arange(n) for n in (g.nz, g.ny, g.nx)), indexing="ij")
    vox = np.stack([x, y, z, np.ones_like(x)], -1).reshape(-1, 4).astype(float)
    world = vox @ np.asarray(g.vox2world).T
    clean = torch.empty(plan.V, dtype=dt, device="cuda")
    plan.backproject(dev(e).to(dt), None, None, clean, None)
    some = False
    for s in rng.permutation(P.M)[:12]:
        off = plan.sample_off[s]
        cand = np.nonzero(val[off:plan.sample_off[s + 1]])[0]
        if cand.size == 0:
            continue
        j = int(rng.choice(cand))
        u, v = P.x0[s] + j % P.w[s], P.y0[s] + j // P.w[s]
        allowed = np.zeros(plan.V, bool)
        for t in ((s - 1, s, s + 1) if f64 else (s,)):  # patches whose packed order holds it
            if not 0 <= t < P.M:
                continue
            A = np.asarray(st[P.stack[t]].pix2world)
            c = A @ np.array([P.x0[t] + 0.5 * (P.w[t] - 1), P.y0[t] + 0.5 * (P.h[t] - 1), P.slice[t], 1.0])
            R = _rotation(th[t])
            pix = np.linalg.solve(A[:, :3], (R.T @ (world - c - th[t, 3:]).T + (c - A[:, 3])[:, None])).T
            sig = st[P.stack[t]].fwhm_mm[2] * synth.FWHM_TO_SIGMA / np.linalg.norm(A[:, 2])
            ru, rv = np.rint(pix[:, 0]) - P.x0[t], np.rint(pix[:, 1]) - P.y0[t]
            w, h = P.w[t], P.h[t]
            if f64:
                hit = np.zeros(len(pix), bool)
                for b in (-1, 0, 1):
                    for a in (-1, 0, 1):
                        hit |= (rv + b) * w + ru + a == off + j - plan.sample_off[t]
                hit &= (ru >= -1) & (ru <= w) & (rv >= -1) & (rv <= h)
            else:
                hit = (np.abs(ru + P.x0[t] - u) <= 1) & (np.abs(rv + P.y0[t] - v) <= 1)
            allowed |= hit & (np.abs(pix[:, 2] - P.slice[t]) <= K * sig * (1 + 1e-6))
        one = np.zeros(plan.N)
        one[off + j] = 1.0
        must = ctx.backproject(th, one).reshape(-1) > 0
        bade = e.copy()
        bade[off + j] = float("nan")
        num = torch.empty_like(clean)
        plan.backproject(dev(bade).to(dt), None, None, num, None)
        bad = np.isnan(host(num))
        some |= bool(must.any())
        assert np.all(bad[must]) and not np.any(bad & ~allowed)
        a, b = host(num)[~bad], host(clean)[~bad]
        assert np.abs(a - b).max() <= (1e-12 if f64 else 1e-5) * np.abs(host(clean)).max()
    assert some


@pytest.mark.parametrize("graph", [False, True])
def test_adjoint_is_itself_again_after_a_value_that_is_not_finite(graph):
    """The slow way that such inputs take does not outlast them: clean inputs give the
    same bits before and after, eagerly and from a replayed graph."""
    g, st, P = _problem(synth.orthogonal_frames([30.0]), 24, 22, 26)
    plan = pvr.Plan([g], [st], [P])
    plan.build(dev(_motion(P.M, 9.0, 1.5).astype(np.float32)))
    e0 = torch.randn(plan.N, device="cuda")
    e = e0.clone()
    num = torch.empty(plan.V, device="cuda")
    run = lambda: plan.backproject(e, None, None, num, None)
    run()
    if graph:
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        G = torch.cuda.CUDAGraph()
        with torch.cuda.graph(G, stream=s):
            run()
            run()
        run = G.replay
    run()
    torch.cuda.synchronize()
    clean = num.clone()
    for value in (float("nan"), float("inf")):
        e[1234] = value
        run()
        torch.cuda.synchronize()
        assert not torch.isfinite(num).all()
        e.copy_(e0)
        run()
        run()
        torch.cuda.synchronize()
        assert torch.equal(num, clean)


def test_a_captured_adjoint_is_itself_again_in_every_replay():
    """One adjoint to a graph, so that every replay prepares where the last one did,
    with an eager one between replays."""
    g, st, P = _problem(synth.orthogonal_frames([30.0]), 24, 22, 26)
    plan = pvr.Plan([g], [st], [P])
    plan.build(dev(_motion(P.M, 9.0, 1.5).astype(np.float32)))
    e0 = torch.randn(plan.N, device="cuda")
    e, other = e0.clone(), e0.clone()
    num, num2 = torch.empty(plan.V, device="cuda"), torch.empty(plan.V, device="cuda")
    plan.backproject(e, None, None, num, None)
    torch.cuda.synchronize()
    clean = num.clone()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    G = torch.cuda.CUDAGraph()
    with torch.cuda.graph(G, stream=s):
        plan.backproject(e, None, None, num, None)
    for value in (float("nan"), float("inf")):
        e[1234] = value
        G.replay()
        torch.cuda.synchronize()
        assert not torch.isfinite(num).all()
        e.copy_(e0)
        for _ in range(3):
            G.replay()
            torch.cuda.synchronize()
            assert torch.equal(num, clean)
            G.replay()
            plan.backproject(other, None, None, num2, None)
            torch.cuda.synchronize()
            assert torch.equal(num, clean) and torch.equal(num2, clean)
