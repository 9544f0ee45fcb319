"""Paths inside the sweep kernels that depend on the line length and the time
step: the interface reduction's lane order on aligned lines and its early end,
the straight-line limiters, and the 4-step scheme's two solves in one launch
(with its fallback to two launches).  Bars: the usual parity bars."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import TOL, GpuProblem, max_rel_err, mixed_rel_err, oracle_run
from tests.test_gpu_parity import _random_problem

pytestmark = pytest.mark.gpu


# aligned lines of 1 to 16 cells per lane on one to four waves (64 ... 4096),
# neighbours of those lengths, and step sizes at which the early end comes
# after few steps (ncfl 1) or never (ncfl 500)
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("n", [64, 128, 256, 512, 1024, 1023, 2048, 4096])
@pytest.mark.parametrize("ncfl", [1.0, 500.0])
def test_aligned_lines_at_small_and_large_steps(prec, variant, n, ncfl):
    p = _random_problem((6, n), "periodic", seed=n, nsteps=3)
    p.h = (1.0 / n, 1.3 / n)
    p.dt = synth.ncfl_dt(ncfl, p.h, 1.0)
    ref = oracle_run(p, prec)
    assert max_rel_err(GpuProblem(p, prec, variant=variant).run(), ref) <= TOL[prec]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("limiter", ["minmod", "mc", "linear", "vanleer"])
@pytest.mark.parametrize("shape,bc", [((33, 256), "periodic"), ((40, 129), "dirichlet"), ((9, 13, 21), "insulating")])
def test_each_limiter_instantiation(prec, limiter, shape, bc):
    p = _random_problem(shape, bc, limiter=limiter, seed=11, nsteps=3)
    err = mixed_rel_err if bc == "dirichlet" else max_rel_err
    for variant in (0, 1):
        assert err(GpuProblem(p, prec, variant=variant).run(), oracle_run(p, prec)) <= TOL[prec]


# two solves in one launch: every capacity, one and several waves per line,
# ragged lines, walls with a source; 10000-cell lines (FP32) do not fit the
# larger tile and take two launches
@pytest.mark.parametrize("prec,n", [(q, n) for q in ("f64", "f32") for n in (17, 64, 128, 250, 512, 1024, 1403, 2048)]
                         + [("f32", 4096), ("f32", 10000)])
@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
def test_four_step_line_lengths(prec, n, bc):
    p = _random_problem((6, n), bc, limiter="vanleer" if n % 2 == 0 else "minmod", seed=n, nsteps=2)
    p.h = (1.0 / n, 1.3 / n)
    p.dt = synth.ncfl_dt(60.0, p.h, 1.0)
    if bc == "dirichlet":
        p.src = 1.0 + 0.2 * synth.smoothed_normal(p.shape, 3, 2.0)
    ref, eref = oracle_run(p, prec, four_step=True, energy=True)
    got, e = GpuProblem(p, prec, four_step=True).run(energy=True)
    err = mixed_rel_err if bc == "dirichlet" else max_rel_err
    assert err(got, ref) <= TOL[prec]
    np.testing.assert_allclose(e, eref, rtol=1e-12 if prec == "f64" else 1e-6, atol=0)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_a_bad_cell_spreads_over_its_line(prec, bad):
    """The early end of the interface reduction needs a finite right-hand
    side: a NaN or infinity reaches every cell of its line, as in the full
    reduction, and raises the status flag."""
    p = _random_problem((8, 1024), "periodic", seed=5, nsteps=1)
    p.h = (1.0 / 1024, 1.3 / 1024)
    p.dt = synth.ncfl_dt(1.0, p.h, 1.0)
    g = GpuProblem(p, prec)
    with torch.cuda.stream(g.stream):
        g.T[3, 700] = bad
    assert not np.isfinite(g.run()[3]).any()
    assert g.g.status()[0] & 1


# grids whose default sweeps store line-contiguous and transpose afterwards:
# the transpose's ragged tiles, walls with a source, both orders, both schemes
@pytest.mark.parametrize("prec,shape,bc,kw", [
    ("f32", (2049, 2101), "periodic", {}),
    ("f32", (2049, 2101), "periodic", {"reverse_order": True}),
    ("f64", (1481, 1500), "dirichlet", {}),
    ("f64", (1481, 1500), "insulating", {"four_step": True}),
])
def test_line_contiguous_store_and_transpose(prec, shape, bc, kw):
    p = _random_problem(shape, bc, seed=9, nsteps=2)
    if bc == "dirichlet":
        p.src = 1.0 + 0.2 * synth.smoothed_normal(shape, 3, 4.0)
    okw = {"reverse": True} if kw.get("reverse_order") else dict(kw)
    ref, eref = oracle_run(p, prec, energy=True, **okw)
    g = GpuProblem(p, prec, **kw)
    T0 = g.T.clone()
    got, e = g.run(energy=True)
    err = mixed_rel_err if bc == "dirichlet" else max_rel_err
    assert err(got, ref) <= TOL[prec]
    np.testing.assert_allclose(e, eref, rtol=1e-12 if prec == "f64" else 1e-7, atol=0)
    # captured and replayed: the same bits
    g.g.set_graphs(True)
    for _ in range(2):
        with torch.cuda.stream(g.stream):
            g.T.copy_(T0)
        assert np.array_equal(g.run(), got)
