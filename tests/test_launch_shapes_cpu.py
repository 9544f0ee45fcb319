"""The default launch shapes over line lengths and counts, on the CPU (a grid
handle needs no device until it steps): every grid that the description check
accepts gets a shape whose lanes hold its lines, within the workgroup limits."""
import ctypes

import pytest
import torch

from paper_1008_0861_amd import binding as asd


def _configs(shape, dtype, **kw):
    d = asd.make_desc(shape, tuple(1.0 / n for n in reversed(shape)), dtype=dtype, **kw)
    nbytes = asd.workspace_bytes(d)
    h = ctypes.c_void_p()
    # the workspace address is only stored and offset here
    asd.check(asd.lib().asd_init_grid(ctypes.byref(d), ctypes.c_void_p(1 << 20), nbytes, None, ctypes.byref(h)))
    out = []
    for axis in range(len(shape)):
        w, l, p, m, io, v = (ctypes.c_int32() for _ in range(6))
        asd.check(asd.lib().asd_get_sweep_config(h, axis, ctypes.byref(w), ctypes.byref(l), ctypes.byref(p), ctypes.byref(m)))
        asd.check(asd.lib().asd_get_sweep_io(h, axis, ctypes.byref(io)))
        asd.check(asd.lib().asd_get_sweep_variant(h, axis, ctypes.byref(v)))
        out.append((w.value, l.value, p.value, m.value, io.value, v.value))
    asd.check(asd.lib().asd_destroy(h))
    return out


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("four", [False, True])
def test_every_accepted_length_has_a_shape(dtype, bc, four):
    es = 4 if dtype == torch.float32 else 8
    longest = 16109 if es == 4 else 4096
    lengths = sorted({3, 5, 16, 17, 63, 64, 65, 127, 128, 129, 511, 512, 513, 1023, 1024, 1025, 1420, 1421, 2047, 2048,
                      2049, 3000, 4095, 4096, 4097, 8191, 8192, 8193, 16109} & set(range(longest + 1)))
    for n in lengths:
        for other in (3, 200, 1030, 4000):
            for shape in ((other, n), (n, other), (3, 4, n)):
                if shape[0] == 3 and len(shape) == 3 and other != 3:
                    continue
                for (wpl, lpw, P, m, io, body), ln in zip(_configs(shape, dtype, bc=bc, four_step=four), reversed(shape)):
                    assert P * m >= ln and P <= 64 * wpl and P <= max(ln, 1)
                    assert 64 * wpl * io * lpw <= (256 if es * m >= 128 else 512 if es * m >= (32 if body else 64) else 1024) \
                        or (es == 4 and not body and 64 * wpl * io * lpw <= 1024)


@pytest.mark.parametrize("shape", [(3, 16385), (3, 20000)])
def test_lines_beyond_the_lds_stay_refused(shape):
    with pytest.raises(asd.AsdError) as e:
        _configs(shape, torch.float32)
    assert e.value.name == "EUNSUPPORTED"
