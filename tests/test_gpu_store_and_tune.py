"""Sweeps whose store is chosen per axis, and tuned 4-step grids: only one axis
line-contiguous, with chi(T), walls, the reverse order and the 4-step scheme's
two launches; shape setters after it; the tuner's choice kept in results."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import TOL, GpuProblem, max_rel_err, mixed_rel_err, oracle_run
from tests.test_gpu_parity import _random_problem

pytestmark = pytest.mark.gpu


# every combination stores in the same order of operations: the transposed
# store's result to the bit where the shape is the same
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("axes", [(0,), (1,), (0, 1)])
@pytest.mark.parametrize("kw", [{}, {"chi_exp": 2.5, "chi_tref": 1.5}, {"reverse_order": True}, {"four_step": True},
                                {"four_step": True, "chi_exp": 2.5, "chi_tref": 1.5}, {"walls": True},
                                {"walls": True, "reverse_order": True}])
def test_line_contiguous_store_per_axis(prec, axes, kw):
    kw = dict(kw)
    bc = "dirichlet" if kw.pop("walls", False) else "periodic"
    p = _random_problem((131, 200), bc, seed=17, nsteps=3, ncfl=10.0)
    if bc == "dirichlet" and "reverse_order" not in kw:
        p.src = 1.0 + 0.2 * synth.smoothed_normal(p.shape, 3, 4.0)
    okw = {"reverse" if k == "reverse_order" else k: v for k, v in kw.items()}
    ref, eref = oracle_run(p, prec, energy=True, **okw)
    err = mixed_rel_err if bc == "dirichlet" else max_rel_err
    got = []
    for store in (False, True):
        g = GpuProblem(p, prec, **kw)
        for a in range(2):
            g.g.set_sweep_config(a, 2, 1)
        if store:
            for a in axes:
                g.g.set_sweep_config(a, 2, 1, split=True)
                # the 4-step scheme's two launches (chi(T)) store transposed
                assert g.g.sweep_config(a).get("split", False) == (not ("four_step" in kw and "chi_exp" in kw))
        T, e = g.run(energy=True)
        assert err(T, ref) <= TOL[prec]
        np.testing.assert_allclose(e, eref, rtol=1e-12 if prec == "f64" else 1e-6, atol=0)
        got.append(T)
    if not ("four_step" in kw and "chi_exp" in kw):  # (there the axis takes its default shape instead)
        assert np.array_equal(*got)


def test_one_axis_by_default():
    """4096 x 1500 FP32: only the axis whose rows are short of a line splits,
    or none; then the shape setters turn it off."""
    p = _random_problem((1100, 4100), "periodic", seed=3, nsteps=2)
    ref = oracle_run(p, "f32")
    g = GpuProblem(p, "f32")
    T0 = g.T.clone()
    assert any(g.g.sweep_config(a).get("split") for a in range(2))
    assert max_rel_err(g.run(), ref) <= TOL["f32"]
    g.g.set_sweep_config(0, 8, 2)
    g.T.copy_(T0)
    torch.cuda.synchronize()
    assert not g.g.sweep_config(0).get("split")
    assert max_rel_err(g.run(), ref) <= TOL["f32"]


@pytest.mark.parametrize("prec,shape,kw", [("f64", (2048, 2048), {"four_step": True}), ("f64", (1403, 300), {"four_step": True}),
                                           ("f32", (1500, 64), {"four_step": True, "chi_exp": 2.5, "chi_tref": 1.5}),
                                           ("f32", (2100, 2100), {})])
def test_tuned_grids(prec, shape, kw):
    p = _random_problem(shape, "periodic", seed=4, nsteps=2, ncfl=10.0)
    g = GpuProblem(p, prec, **kw)
    T0 = g.T.clone()
    with torch.cuda.stream(g.stream):
        g.g.tune(p.dt, reps=3)
    assert torch.equal(g.T, T0)
    c = [g.g.sweep_config(a) for a in range(2)]
    if shape == (2048, 2048):
        # one launch per direction: what two solves in two launches cost is
        # timed as such (the shapes of 8 waves per line take two)
        assert all(q["variant"] == 0 and q["io"] == 1 and q["wpl"] <= 4 for q in c), c
    ref = oracle_run(p, prec, **kw)
    assert max_rel_err(g.run(), ref) <= TOL[prec]
    for a, q in enumerate(c):  # the round trip through the setters
        g.g.set_sweep_config(a, q["wpl"], q["lpw"], q["io"], q["variant"], split=q.get("split", False))
    assert [g.g.sweep_config(a) for a in range(2)] == c
    g.T.copy_(T0)
    torch.cuda.synchronize()
    assert max_rel_err(g.run(), ref) <= TOL[prec]


@pytest.mark.parametrize("kw", [{}, {"four_step": True}, {"four_step": True, "chi_exp": 2.0}])
def test_single_sweeps_timed_leave_T(kw):
    p = _random_problem((2100, 2100), "periodic", seed=6, nsteps=1)
    g = GpuProblem(p, "f32", **kw)
    T0 = g.T.clone()
    torch.cuda.synchronize()
    with torch.cuda.stream(g.stream):
        g.g.bench_sweep(0, p.dt, 0)
        for a in range(2):
            g.g.bench_sweep(a, p.dt, 2)
    g.stream.synchronize()
    assert torch.equal(g.T, T0)
