"""The explicit step's instantiations (constant chi, per-cell chi, everything
at run time) and its 3-D march: rows and planes per wave change with the size
(two rows below 2^19 cells and in FP64, 2 to 32 planes), at ragged edges of the
62-column, row and plane blocks."""
import numpy as np
import pytest

import synth
from tests.gpu_util import TOL, GpuProblem, max_rel_err, mixed_rel_err, oracle_run
from tests.test_gpu_parity import _random_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("shape", [(3, 3, 3), (2, 5, 62), (33, 6, 63), (5, 7, 125), (67, 130, 64), (200, 61, 64), (37, 64)])
@pytest.mark.parametrize("mode", ["const", "cell", "walls-source", "minmod-cell"])
def test_explicit_modes(prec, shape, mode):
    bc = "dirichlet" if mode == "walls-source" else "insulating" if (2 in shape or mode == "cell") else "periodic"
    p = _random_problem(shape, bc, limiter="minmod" if "minmod" in mode else "vanleer", per_cell_chi="cell" in mode,
                        seed=sum(shape), nsteps=3)
    p.dt = 0.2 * min(p.h) ** 2 / (1.0 if p.chi is None else float(p.chi.max()))
    if mode == "walls-source":
        p.src = 1.0 + 0.2 * synth.smoothed_normal(shape, 3, 2.0)
    ref, eref = oracle_run(p, prec, scheme="ex", energy=True)
    got, e = GpuProblem(p, prec).run(scheme="ex", energy=True)
    err = mixed_rel_err if bc == "dirichlet" else max_rel_err
    assert err(got, ref) <= TOL[prec]
    np.testing.assert_allclose(e, eref, rtol=1e-12 if prec == "f64" else 1e-6, atol=0)
