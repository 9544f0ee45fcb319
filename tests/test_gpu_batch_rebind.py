"""Problems set again between step calls that are not waited for: the tables
are rewritten only when the kernels in flight have read them."""
import pytest
import torch

import synth
from paper_1008_0861_amd import binding as asd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 2])
def test_set_problem_between_calls_in_flight(mode):
    import ctypes
    probs = synth.batch_problems(nprob=6, master_seed=5, sides=[64, 129, 256], nsteps=4)
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    st = torch.cuda.Stream()

    def batch(states):
        return asd.Batch([dict(shape=p.shape, h=p.h, chi_par=p.chi_par, dt=p.dt, T=t, bx=dev(p.b[0]), by=dev(p.b[1]))
                          for p, t in zip(probs, states)], dtype=torch.float64, stream=st)

    with torch.cuda.stream(st):
        one, two = [[dev(p.T0 + k) for p in probs] for k in range(2)]
        ref = []
        for states in ([t.clone() for t in one], [t.clone() for t in two]):
            b = batch(states)
            b.step(40, mode)
            st.synchronize()
            ref.append(states)
        b = batch(one)
        b.step(40, mode)
        for i, t in enumerate(two):  # while the first call runs
            it = b.problems[i]
            asd.check(asd.lib().asd_batch_set_problem(b.handle, i, *(ctypes.c_void_p(v.data_ptr()) for v in (t, it["bx"], it["by"])),
                                                      float(it["dt"])))
        b.step(40, mode)
    st.synchronize()
    for got, want in zip(one + two, ref[0] + ref[1]):
        assert torch.equal(got, want)
