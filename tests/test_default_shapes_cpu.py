"""Which launch shapes are the defaults, on the CPU (handles need no device
until they step): one case on each side of the measured rules."""
import ctypes

import pytest
import torch

from paper_1008_0861_amd import binding as asd

F32, F64 = torch.float32, torch.float64
FACE, CELL = 0, 1


def batch_body(dtype, bc):
    d = (asd.Desc * 2)()
    for i, shape in enumerate([(64, 300), (130, 512)]):
        d[i] = asd.make_desc(shape, tuple(1.0 / n for n in reversed(shape)), bc=bc, dtype=dtype)
    n, h, v = ctypes.c_size_t(), ctypes.c_void_p(), ctypes.c_int32()
    asd.check(asd.lib().asd_batch_workspace_bytes(d, 2, ctypes.byref(n)))
    # the workspace address is only stored and offset here
    asd.check(asd.lib().asd_batch_init(d, 2, ctypes.c_void_p(1 << 20), n.value, None, ctypes.byref(h)))
    asd.check(asd.lib().asd_batch_get_variant(h, ctypes.byref(v)))
    asd.check(asd.lib().asd_batch_destroy(h))
    return v.value


@pytest.mark.parametrize("dtype,bc,body", [(F32, "periodic", CELL), (F32, "insulating", CELL), (F32, "dirichlet", FACE),
                                           (F64, "periodic", FACE), (F64, "dirichlet", FACE)])
def test_batch_body(dtype, bc, body):
    assert batch_body(dtype, bc) == body


def sweep_shape(shape, dtype, axis=0, **kw):
    """(body, waves per line, lines per workgroup) of one sweep of a fresh grid."""
    d = asd.make_desc(shape, tuple(1.0 / n for n in reversed(shape)), dtype=dtype, **kw)
    h = ctypes.c_void_p()
    asd.check(asd.lib().asd_init_grid(ctypes.byref(d), ctypes.c_void_p(1 << 20), asd.workspace_bytes(d), None, ctypes.byref(h)))
    w, l, p, m, v = (ctypes.c_int32() for _ in range(5))
    asd.check(asd.lib().asd_get_sweep_config(h, axis, ctypes.byref(w), ctypes.byref(l), ctypes.byref(p), ctypes.byref(m)))
    asd.check(asd.lib().asd_get_sweep_variant(h, axis, ctypes.byref(v)))
    asd.check(asd.lib().asd_destroy(h))
    return v.value, w.value, l.value


@pytest.mark.parametrize("shape,dtype,expect", [
    ((1024, 1024), F32, (CELL, 2, 4)),
    ((1120, 1120), F32, (CELL, 2, 2)),   # whole half lines: the fourth line costs a third more
    ((1100, 1100), F32, (CELL, 2, 4)),   # rows start anywhere: whole pieces
    ((1130, 1130), F32, (FACE, 2, 4)),   # ... and one workgroup of four lines per CU with cell slots
    ((937, 1403), F32, (CELL, 2, 4)),    # four lines are all that a CU gets
    ((1403, 1403), F32, (FACE, 2, 4)),
    ((1344, 1344), F32, (CELL, 2, 2)),
    ((1520, 1520), F32, (CELL, 2, 2)),   # three workgroups of cell slots per CU
    ((1536, 1536), F32, (FACE, 2, 2)),   # two
    ((1792, 1792), F32, (FACE, 2, 4)),
    ((2000, 2000), F32, (FACE, 2, 2)),   # rows on half lines
    ((2048, 2048), F32, (FACE, 2, 4)),
    ((2000, 1200), F32, (FACE, 2, 2)),   # eight lines per CU, six held with cell slots
    ((2320, 1280), F32, (CELL, 2, 2)),   # ten lines: the second round is nearly full
    ((1935, 1936), F32, (FACE, 2, 2)),   # rows one element short of a half line
    ((512, 512), F64, (CELL, 1, 2)),
    ((1649, 432), F64, (CELL, 1, 4)),
    ((3000, 500), F64, (FACE, 1, 4)),
    ((512, 1999), F64, (FACE, 4, 1)),
    ((768, 768), F64, (FACE, 2, 2)),
    ((60, 600), F64, (CELL, 2, 1)),
    ((896, 896), F64, (CELL, 2, 2)),
    ((1100, 1100), F64, (FACE, 2, 2)),
    ((1200, 1200), F64, (FACE, 4, 1)),
    ((1403, 1403), F64, (FACE, 2, 2)),
    ((1536, 1536), F64, (FACE, 4, 1)),
    ((1920, 1920), F64, (FACE, 2, 2)),
    ((2048, 2048), F64, (FACE, 4, 1)),
    ((300, 3000), F64, (FACE, 4, 1)),
    ((100, 3000), F64, (FACE, 8, 1)),
    ((64, 64, 64), F32, (CELL, 1, 4)),
    ((100, 100, 100), F32, (FACE, 1, 4)),
    ((128, 128, 128), F32, (CELL, 1, 4)),
])
def test_sweep_shape(shape, dtype, expect):
    assert sweep_shape(shape, dtype) == expect


@pytest.mark.parametrize("shape,dtype,kw,expect", [
    ((1536, 1536), F32, {}, (FACE, 4, 2)),
    ((1200, 1200), F32, {}, (FACE, 4, 2)),
    ((937, 1403), F32, {}, (FACE, 2, 4)),
    ((1500, 1500), F32, {}, (FACE, 2, 4)),
    ((1536, 1536), F64, {}, (FACE, 4, 1)),
    ((1403, 1403), F64, {}, (FACE, 4, 1)),
    ((256, 4096), F64, {}, (FACE, 4, 1)),
    ((128, 128, 128), F32, {}, (FACE, 1, 8)),
    # chi(T) rebuilds the coefficients between the solves: two launches, the one-solve shapes
    ((1536, 1536), F32, dict(chi_exp=2.5, chi_tref=1.5), (FACE, 2, 2)),
    ((1536, 1536), F64, dict(chi_exp=2.5, chi_tref=1.5), (FACE, 4, 1)),
    ((128, 128, 128), F32, dict(chi_exp=2.5, chi_tref=1.5), (CELL, 1, 4)),
])
def test_sweep_shape_four_step(shape, dtype, kw, expect):
    assert sweep_shape(shape, dtype, four_step=True, **kw) == expect
