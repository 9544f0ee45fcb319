"""The differentiable steps keep the states for the backward only where one can
follow."""
import numpy as np
import pytest
import torch

from paper_1008_0861_amd import autograd, binding
from tests.test_gpu_adjoint import _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,states", [("grad", True), ("chi", True), ("plain", False), ("no_grad", False)])
def test_forward_stores_states_only_for_a_backward(mode, states):
    b, T0, chi, h, dt = _problem((37, 50), 21)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        t0, c, *bb = (torch.from_numpy(np.ascontiguousarray(a)).double().cuda() for a in (T0, chi, *b))
        g = binding.Grid(T0.shape, h, dtype=torch.float64, chi_par=float(chi.max()), per_cell_chi=True, stream=st)
        g.set_b(*bb)
    st.synchronize()
    seen, run = [], g.adjoint_forward
    g.adjoint_forward = lambda *a, **kw: seen.append(kw["states"]) or run(*a, **kw)
    want = autograd.semi_implicit_steps(t0.clone().requires_grad_(), c, g, dt, 6, 6)
    t0.requires_grad_(mode in ("grad", "no_grad"))
    c.requires_grad_(mode == "chi")
    with torch.set_grad_enabled(mode != "no_grad"):
        T = autograd.semi_implicit_steps(t0, c, g, dt, 6, 6)
    assert seen == [True, states] and T.requires_grad == states
    assert torch.equal(T.detach(), want.detach())
    if states:
        T.sum().backward()
        assert torch.isfinite((t0 if mode == "grad" else c).grad).all()
