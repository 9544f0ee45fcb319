"""What the shape getters report and the setters restore, on the CPU (a grid
handle needs no device until it steps): the store of large 2-D grids, and the
bodies of 4-step grids, whose two solves share a launch on face slots only."""
import ctypes

import pytest
import torch

from paper_1008_0861_amd import binding as asd

F32, F64 = torch.float32, torch.float64
FACE, CELL = 0, 1


class Handle(asd.Grid):
    """A grid without device memory."""

    def __init__(self, shape, dtype, **kw):
        self.shape = shape
        d = asd.make_desc(shape, tuple(1.0 / n for n in reversed(shape)), dtype=dtype, **kw)
        self.handle = ctypes.c_void_p()
        # the workspace address is only stored and offset here
        asd.check(asd.lib().asd_init_grid(ctypes.byref(d), ctypes.c_void_p(1 << 20), asd.workspace_bytes(d), None,
                                          ctypes.byref(self.handle)))

    def configs(self):
        return [self.sweep_config(a) for a in range(len(self.shape))]

    def restore(self, configs):
        for a, c in enumerate(configs):
            self.set_sweep_config(a, *(c[k] for k in ("wpl", "lpw", "io", "variant")), split=c.get("split", False))


@pytest.mark.parametrize("shape,dtype,kw,split", [
    ((4096, 4096), F32, {}, True), ((2500, 2500), F32, {}, True), ((2500, 2500), F32, dict(bc="dirichlet"), True),
    ((1500, 1500), F64, {}, True), ((2500, 2500), F64, dict(four_step=True), True), ((3000, 3000), F32, dict(four_step=True), True),
    ((2048, 2048), F32, {}, False), ((1024, 1024), F64, {}, False), ((2500, 2500), F64, dict(four_step=True, chi_exp=2.0), False),
])
def test_shapes_and_store_round_trip(shape, dtype, kw, split):
    g = Handle(shape, dtype, **kw)
    was = g.configs()
    assert [c.get("split", False) for c in was] == [split] * 2
    if split:  # one line per workgroup, the shape that runs
        assert all(c["lpw"] == 1 for c in was)
    g.set_sweep_config(0, 8, 1)
    assert g.sweep_config(0)["wpl"] == 8 and "split" not in g.sweep_config(0)
    g.restore(was)
    assert g.configs() == was
    other = Handle(shape, dtype, **kw)
    other.restore(was)
    assert other.configs() == was


def test_store_arguments():
    g = Handle((64, 64), F64)
    s = ctypes.c_int32(7)
    lib = asd.lib()
    assert lib.asd_get_sweep_store(g.handle, 0, ctypes.byref(s)) == 0 and s.value == 0
    assert lib.asd_set_sweep_store(g.handle, 0, 1) == 0
    assert lib.asd_get_sweep_store(g.handle, 0, ctypes.byref(s)) == 0 and s.value == 1
    assert lib.asd_set_sweep_store(g.handle, 0, 2) == -1 and lib.asd_set_sweep_store(g.handle, 2, 0) == -1
    assert lib.asd_get_sweep_store(g.handle, 0, None) == -1
    with pytest.raises(asd.AsdError) as e:
        asd.check(lib.asd_set_sweep_store(Handle((8, 8, 8), F64).handle, 0, 1))
    assert e.value.name == "EUNSUPPORTED"


@pytest.mark.parametrize("shape", [(1024, 1024), (200, 300), (64, 64, 64)])
@pytest.mark.parametrize("dtype", [F32, F64])
def test_four_step_reports_the_body_that_runs(shape, dtype):
    g = Handle(shape, dtype, four_step=True)
    # one launch for both solves: face slots
    assert all(c["variant"] == FACE and c["io"] == 1 for c in g.configs())
    for a in range(len(shape)):
        c = g.sweep_config(a)
        g.set_sweep_config(a, c["wpl"], 1, 1, CELL)
    assert all(c["variant"] == CELL and c["lpw"] == 1 for c in g.configs())


def test_four_step_reports_the_lines_per_workgroup_that_fit():
    g = Handle((1024, 1024), F64, four_step=True)
    g.set_sweep_config(0, 2, 4)  # 512 threads: the two-solve launch takes 256
    assert g.sweep_config(0)["lpw"] == 2
    assert Handle((1024, 1024), F64).sweep_config(0)["lpw"] >= 1
