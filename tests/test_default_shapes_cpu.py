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
