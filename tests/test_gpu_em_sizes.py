"""The patch classification at the edges of its launches: problems of one
patch, of about 64 and 256 (one and four wavefronts), of about one patch a lane
of the full workgroup, and of what its LDS copy holds and one more.  Random
residuals, a fifth of the patches with ten times the noise, against the FP64
oracle.  Bar: a potential is right to 1e-6 (sums of FP32 posteriors); a weight
follows it by at most 1/4 of the exponent's change, 2 (d / sd) (1 / sd) 1e-6
with sd >= 1e-3 and d / sd <= 4 where the weight is neither 0 nor 1: 2e-3."""
import numpy as np
import pytest
import torch

from oracle import recon
from paper_1611_07289_amd import pvr, synth
from tests.test_gpu_parity import dev, host

pytestmark = pytest.mark.gpu

BAR = 2e-3


@pytest.mark.parametrize("sizes", [(1,), (2,), (3, 1), (63,), (64,), (65, 3), (255,), (256, 64),
                                   (257,), (1023,), (1025, 70), (4097,), (12288,), (12289,)])
def test_weights(sizes):
    rng = np.random.default_rng(sum(sizes))
    P = synth.tiny_problem()
    grids, stacks, pats = [], [], []
    for n in sizes:
        st = P.stacks[0]
        cols = [np.zeros(n), rng.integers(2, 6, n), rng.integers(8, 20, n),
                rng.integers(8, 20, n), np.full(n, 4), np.full(n, 3)]
        grids.append(P.grid)
        stacks.append([st])
        pats.append(synth.Patches(*[np.asarray(c, np.int32) for c in cols]))
    plan = pvr.Plan(grids, stacks, pats)
    plan.build(torch.zeros(plan.M, 6, device="cuda"))
    y = rng.uniform(100, 900, plan.N).astype(np.float32)
    loud = np.repeat(rng.random(plan.M) < 0.2, 12)
    e = (rng.normal(size=plan.N) * np.where(loud, 30.0, 3.0) * rng.uniform(0.5, 1.5, plan.N)).astype(np.float32)
    em = plan.em_state()
    p, pbar, W = (torch.empty(n, device="cuda") for n in (plan.N, plan.M, plan.M))
    plan.robust_weights(dev(e), dev(y), em, p, pbar, W, flags=pvr.PVR_EM_INIT)
    states = pvr.Plan.read_em(em)
    W, s0 = host(W), 0
    val = np.ones(plan.N, bool)  # patches well inside the grid
    for st, n in zip(states, sizes):
        j = slice(12 * s0, 12 * (s0 + n))
        ref = recon.robust_weights(np.where(val[j], e[j], 0).astype(np.float64), y[j].astype(np.float64),
                                   val[j], recon.EMState(), np.repeat(np.arange(n), 12), n)
        Wr, pi, new = ref[2], ref[3], ref[4]
        near = np.abs(pi - 0.5) <= BAR
        w = W[s0:s0 + n]
        assert np.array_equal((w > 0)[~near], (Wr > 0)[~near])
        assert np.all(np.abs(w - Wr)[~near] <= BAR)
        if not near.any():
            assert st.n_excluded == int(np.sum((Wr == 0)))
            assert st.sigma2 == pytest.approx(new.sigma2, rel=BAR)
            assert st.c == pytest.approx(new.c, rel=BAR)
        s0 += n
