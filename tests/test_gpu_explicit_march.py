"""The 3-D explicit step's march along z over many planes: 4 rows per wave in
FP32 on grids of 2^21 cells and more, 2 otherwise, marches of 8, 16 and 32
planes (and, with chi(T), of counts in between) whose last block is shorter,
for every chi form and limiter instantiation."""
import numpy as np
import pytest

import synth
from tests.gpu_util import TOL, GpuProblem, max_rel_err, mixed_rel_err, oracle_run
from tests.test_gpu_parity import _random_problem

pytestmark = pytest.mark.gpu

# (rows, planes) with a constant or per-cell chi; a wave covers 62 columns, and
# the planes are the most of 2 ... 32 that leave 3072 waves
F32 = [((410, 262, 20), 4, 8), ((780, 258, 11), 4, 16), ((1970, 201, 6), 4, 32), ((820, 62, 5), 2, 8)]
F64 = [((820, 62, 5), 2, 8), ((3190, 62, 5), 2, 32)]


@pytest.mark.parametrize("prec,shape,rows,planes", [("f32", *c) for c in F32] + [("f64", *c) for c in F64])
@pytest.mark.parametrize("mode", ["const-vanleer", "cell-mc", "walls-source-minmod", "of-T-linear"])
def test_long_march(prec, shape, rows, planes, mode):
    nz, ny, nx = shape
    cols = -(-nx // 62) * -(-ny // rows)
    assert (rows == 4) == (prec == "f32" and nx * ny * nz >= 1 << 21)
    assert cols * -(-nz // planes) >= 3072 and (planes == 32 or cols * -(-nz // (2 * planes)) < 3072)
    assert nz % planes and nz > 2 * planes
    bc = "dirichlet" if "walls" in mode else "insulating" if "cell" in mode else "periodic"
    p = _random_problem(shape, bc, limiter=mode.split("-")[-1], per_cell_chi="cell" in mode, seed=nz, nsteps=2)
    p.dt = 0.1 * min(p.h) ** 2 / (1.0 if p.chi is None else float(p.chi.max()))
    if "source" in mode:
        p.src = 1.0 + 0.2 * synth.smoothed_normal(shape, 3, 2.0)
    if "of-T" in mode:
        from oracle import oracle
        from tests.gpu_util import rounded
        b, T0, _ = rounded(p, prec)
        o = oracle.OracleGrid(b, p.h, bc=p.bc, limiter=p.limiter, chi_par=p.chi_par, chi_exp=2.5, chi_tref=2.0)
        ref, eref = o.step_explicit(T0, p.dt, 2, energy=True)
        got, e = GpuProblem(p, prec, chi_exp=2.5, chi_tref=2.0).run(scheme="ex", energy=True)
    else:
        ref, eref = oracle_run(p, prec, scheme="ex", energy=True)
        got, e = GpuProblem(p, prec).run(scheme="ex", energy=True)
    err = mixed_rel_err if bc == "dirichlet" else max_rel_err
    assert err(got, ref) <= TOL[prec]
    np.testing.assert_allclose(e, eref, rtol=1e-12 if prec == "f64" else 1e-6, atol=0)
