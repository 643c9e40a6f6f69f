"""Stream ordering of the registration on each of its routes.  Up to 256 steps central
differences move all patches in step, on the call's stream alone; beyond, and with
the exact gradient on small plans, a workgroup runs each patch, those that read the
volume's y-fastest copy on the plan's second stream, joined back before the call
returns.  A copy taken on the caller's stream right after the call equals the final
values, for patches of both layouts (the 32^3 workload's sagittal stack runs its rows
along voxel y)."""
import numpy as np
import pytest
import torch

from paper_1611_07289_amd import pvr, synth
from tests._gpu import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_iter", [40, 257])
@pytest.mark.parametrize("exact,psf", [(False, pvr.PVR_PSF_GAUSSIAN), (True, pvr.PVR_PSF_GAUSSIAN),
                                       (False, pvr.PVR_PSF_SINC)])
def test_results_are_ordered_on_the_call_stream(exact, psf, max_iter):
    P = synth.tiny_problem()
    print(f"[gpu] registration order exact={exact} psf={psf} steps={max_iter}", flush=True)
    th0 = (P.theta_true + synth.random_motion(P.M, 3.0, 1.0, 7)).astype(np.float32)
    plan = pvr.Plan.from_problems([P])
    plan.set_psf(psf)
    plan.build(dev(P.theta_true, torch.float32))
    X = dev(P.x_true.reshape(-1).astype(np.float32))
    y = torch.empty(plan.N, device="cuda")
    plan.simulate(X, y_sim=y)
    plan.build(dev(th0))
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        tt = dev(th0)
        ncc = torch.zeros(plan.M, dtype=torch.float32, device="cuda")
        plan.register(X, y, tt, ncc, params=pvr.RegParams.make(exact=exact, max_iter=max_iter))
        snap_t, snap_n = tt.clone(), ncc.clone()
    s.synchronize()
    torch.cuda.synchronize()
    assert torch.equal(snap_t, tt)
    assert torch.equal(snap_n, ncc)
    moved = (tt.cpu().numpy() != th0).any(1)
    for st in range(len(P.stacks)):
        assert moved[P.patches.stack == st].any(), st
