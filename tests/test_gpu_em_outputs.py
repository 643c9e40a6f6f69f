"""The potentials of the robust weights are an output the caller may leave out: the
posteriors, the patch weights and the state do not depend on it."""
import numpy as np
import pytest
import torch

from paper_1611_07289_amd import pvr, synth
from _gpu import dev, host

pytestmark = pytest.mark.gpu


def test_weights_without_the_potentials():
    P = synth.tiny_problem()
    plan = pvr.Plan.from_problems([P])
    plan.build(dev(P.theta_true.astype(np.float32)))
    rng = np.random.default_rng(5)
    y = dev((400.0 + 50.0 * rng.normal(size=P.N)).astype(np.float32))
    e = dev((30.0 * rng.normal(size=P.N)).astype(np.float32))
    out = []
    for with_pbar in (True, False):
        em, p = plan.em_state(), torch.full((plan.N,), float("nan"), device="cuda")
        pbar = torch.full((plan.M,), float("nan"), device="cuda") if with_pbar else None
        W = torch.full((plan.M,), float("nan"), device="cuda")
        for flags in (pvr.PVR_EM_INIT, 0):
            plan.robust_weights(e, y, em, p, pbar, W, flags=flags)
        s = pvr.Plan.read_em(em)[0]
        out.append((host(p), host(W), [s.m, s.sigma2, s.c]))
        if with_pbar:
            assert np.isfinite(host(pbar)).all()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    assert out[0][2] == out[1][2]
