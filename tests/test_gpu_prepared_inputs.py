"""The adjoint inputs that the robust weights prepare (PVR_EM_PREP_ADJOINT) are
taken only where they still describe the call's residuals and posteriors: not
after a back-projection of other buffers, a simulation by tiles, or the launch
of a captured graph, which all leave other values behind, and not across the
capture of a stream, whose calls have not run.  Every case is compared bit for
bit with the same calls without the flag."""
import pytest
import torch

from paper_1611_07289_amd import pvr, synth
from _gpu import dev

pytestmark = pytest.mark.gpu

BASE = pvr.PVR_EM_INIT | pvr.PVR_EM_RESID_FRESH


class Bufs:
    def __init__(self, plan):
        f = lambda n: torch.zeros(n, device="cuda")
        self.e, self.p, self.pbar, self.W = f(plan.N), f(plan.N), f(plan.M), f(plan.M)
        self.num, self.den, self.em = f(plan.V), f(plan.V), plan.em_state()


@pytest.fixture(scope="module")
def setup():
    P = synth.tiny_problem()
    plan = pvr.Plan.from_problems([P])
    plan.build(dev(P.theta_true, torch.float32))
    X = dev(P.x_true.reshape(-1))
    y = torch.empty(plan.N, device="cuda")
    plan.simulate(X, y_sim=y)
    y += 5.0 * torch.randn(plan.N, generator=torch.Generator("cuda").manual_seed(1), device="cuda")
    return plan, 0.9 * X, y


def _weights(plan, b, X, y, flags):
    plan.simulate(X, y_obs=y, resid=b.e)
    plan.robust_weights(b.e, y, b.em, b.p, b.pbar, b.W, flags)


def _other_buffers(plan, b, X, y):
    e2, p2 = torch.rand_like(b.e), torch.rand_like(b.p)
    plan.backproject(e2, p2, b.W, torch.empty_like(b.num), torch.empty_like(b.den))


def _tiles(plan, b, X, y):
    plan.set_tiles(16, 16)
    plan.simulate(1.05 * X, y_obs=y, resid=b.e)
    plan.set_tiles(0, 0)


def _graph(plan, b, X, y):
    c = Bufs(plan)
    _weights(plan, c, X, y, BASE)  # the graph continues from an EM state
    plan.simulate(X, y_obs=y, resid=b.e)
    g = pvr.SRGraph(plan, 1.1 * X, torch.empty_like(X), y, c.e, c.p, c.pbar, c.W, c.num, c.den, c.em,
                    iters=2)
    plan.robust_weights(b.e, y, b.em, b.p, b.pbar, b.W, b.flags)
    g.launch()
    torch.cuda.synchronize()
    g.close()


@pytest.mark.parametrize("between", [_other_buffers, _tiles, _graph])
def test_prepared_inputs_do_not_outlive_their_values(setup, between):
    plan, X, y = setup
    out = []
    for flags in (BASE, BASE | pvr.PVR_EM_PREP_ADJOINT):
        b = Bufs(plan)
        b.flags = flags
        _weights(plan, b, X, y, flags)
        between(plan, b, X, y)
        plan.backproject(b.e, b.p, b.W, b.num, b.den)
        torch.cuda.synchronize()
        out.append((b.num, b.den))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert float(out[0][0].abs().max()) > 0


def _captured(fn):
    g = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        fn()
    torch.cuda.synchronize()
    return g


def test_a_captured_gather_prepares_its_own_inputs(setup):
    """Weights eagerly, the back-projection alone in a graph: a replay takes the
    residuals that are there then."""
    plan, X, y = setup
    b = Bufs(plan)
    _weights(plan, b, X, y, BASE | pvr.PVR_EM_PREP_ADJOINT)
    plan.backproject(b.e, b.p, b.W, b.num, b.den)  # the index
    _weights(plan, b, X, y, BASE | pvr.PVR_EM_PREP_ADJOINT)
    g = _captured(lambda: plan.backproject(b.e, b.p, b.W, b.num, b.den))
    for k in (1.0, 2.0, 3.0):
        b.e.mul_(k)
        g.replay()
        torch.cuda.synchronize()
        num, den = b.num.clone(), b.den.clone()
        plan.backproject(b.e, torch.empty_like(b.p).copy_(b.p), b.W, b.num, b.den)
        assert torch.equal(num, b.num) and torch.equal(den, b.den)


def test_captured_weights_prepare_nothing_for_an_eager_gather(setup):
    plan, X, y = setup
    b, c = Bufs(plan), Bufs(plan)
    _weights(plan, b, X, y, BASE)
    plan.backproject(b.e, b.p, b.W, b.num, b.den)
    _weights(plan, c, X, y, BASE)
    g = _captured(lambda: plan.robust_weights(b.e, y, c.em, b.p, c.pbar, c.W,
                                              BASE | pvr.PVR_EM_PREP_ADJOINT))
    e, p = b.e, b.p
    _other_buffers(plan, c, X, y)
    plan.backproject(e, p, b.W, c.num, c.den)
    torch.cuda.synchronize()
    assert torch.equal(c.num, b.num) and torch.equal(c.den, b.den)
    del g


def test_an_index_recorded_in_a_capture_is_not_an_eager_call_s(setup):
    """The first back-projection after a build, captured and never replayed: the
    eager one that follows builds the index it needs."""
    plan, X, y = setup
    b = Bufs(plan)
    _weights(plan, b, X, y, BASE)
    plan.backproject(b.e, b.p, b.W, b.num, b.den)
    P = synth.tiny_problem()
    other = pvr.Plan.from_problems([P])
    other.build(dev(P.theta_true, torch.float32))
    num, den = torch.empty_like(b.num), torch.empty_like(b.den)
    g = _captured(lambda: other.backproject(b.e, b.p, b.W, num, den))
    other.backproject(b.e, b.p, b.W, num, den)
    torch.cuda.synchronize()
    assert torch.equal(num, b.num) and torch.equal(den, b.den)
    g.replay()
    torch.cuda.synchronize()
    assert torch.equal(num, b.num) and torch.equal(den, b.den)
