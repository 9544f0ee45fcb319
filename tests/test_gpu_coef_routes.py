"""The face coefficients' two kernels (a thread per cell; 32 x 32 tiles through
LDS) on both sides of each rule that chooses between them: grids of up to 2^17
cells in 2-D and 2^18 in 3-D (2^19 with chi(T)), rows shorter than 16 cells, and with chi(T) lines of
at most 48 bytes, each with periodic and wall faces."""
import pytest

from tests.gpu_util import TOL, GpuProblem, max_rel_err, mixed_rel_err, oracle_run
from tests.test_gpu_parity import _random_problem

pytestmark = pytest.mark.gpu

SHAPES = [(2, 2), (3, 3), (33, 31), (362, 363), (361, 364), (64, 64, 64), (65, 64, 64), (300, 31, 15), (300, 31, 16),
          (65, 33, 64)]
OF_T = [(3, 3), (64, 33), (724, 725), (723, 724), (100, 80, 65), (82, 80, 81), (12, 230, 230), (13, 230, 230),
        (6, 320, 310), (7, 320, 310), (230, 12, 230)]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("bc", ["periodic", "insulating", "dirichlet"])
@pytest.mark.parametrize("shape", SHAPES)
def test_constant_and_cell_chi(prec, bc, shape):
    if 2 in shape and bc == "periodic":
        pytest.skip("a periodic axis needs three cells")
    p = _random_problem(shape, bc, per_cell_chi=shape[0] % 2 == 1, chi_perp=0.0 if shape[0] % 2 else 1e-2,
                        seed=sum(shape), nsteps=2)
    err = mixed_rel_err if bc == "dirichlet" else max_rel_err
    assert err(GpuProblem(p, prec).run(), oracle_run(p, prec)) <= TOL[prec]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("bc", ["periodic", "insulating"])
@pytest.mark.parametrize("shape", OF_T)
def test_chi_of_T(prec, bc, shape):
    p = _random_problem(shape, bc, seed=sum(shape), ncfl=10.0, nsteps=2)
    ref = oracle_run(p, prec, chi_exp=2.5, chi_tref=1.5)
    got = GpuProblem(p, prec, chi_exp=2.5, chi_tref=1.5).run()
    assert max_rel_err(got, ref) <= TOL[prec]
