"""The adjoint pair that keeps every state of at most two segments against
the pair that recomputes them, bit for bit, twice from one workspace."""
import numpy as np
import pytest
import torch

from tests.test_gpu_adjoint import AdjGrid, _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("nsteps,k", [(1, 1), (2, 1), (3, 1), (12, 12), (12, 50), (12, 6), (7, 4), (13, 4), (0, 3)])
def test_stored_states_give_the_recomputed_gradients(prec, nsteps, k):
    b, T0, chi, h, dt = _problem((37, 50), 21)
    ag = AdjGrid(b, chi, h, prec)
    rng = np.random.default_rng(5)
    with torch.cuda.stream(ag.stream):
        t0 = torch.from_numpy(T0).to(ag.dt).cuda()
        runs = []
        for states in (False, True):
            T = t0.clone()
            ag.g.set_field("T", T)
            ws = ag.g.adjoint_workspace(nsteps, k).fill_(0xAB)
            ag.g.adjoint_forward(dt, nsteps, k, ws, states=states)
            T.mul_(2.0)  # the caller's T is its own again after the forward
            runs.append((T, ws))
        for _ in range(2):
            lam = torch.from_numpy(rng.standard_normal(T0.shape)).to(ag.dt).cuda()
            a, c = (ag.g.adjoint_stored(dt, nsteps, k, ws, lam, states=s) for s, (_, ws) in zip((False, True), runs))
            assert torch.equal(a[0], c[0]) and torch.equal(a[1], c[1])
    assert torch.equal(runs[0][0], runs[1][0])
