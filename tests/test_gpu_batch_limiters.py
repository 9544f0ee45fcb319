"""The batch kernels' instantiations: every limiter with and without T = 0
walls, on both tile bodies, at each per-lane capacity, persistent and grouped,
against the oracle (lines of 9 to 300 cells: ragged, aligned, two per wave)."""
import dataclasses

import numpy as np
import pytest
import torch

import synth
from paper_1008_0861_amd import binding as asd
from tests.gpu_util import DT, TOL, max_rel_err, mixed_rel_err, oracle_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("limiter", ["vanleer", "minmod", "mc", "linear"])
@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
def test_limiter_instantiations(prec, limiter, bc):
    probs = synth.batch_problems(nprob=5, master_seed=31, sides=np.array([9, 33, 64, 128, 300]), nsteps=2)
    probs = [dataclasses.replace(p, bc=bc, limiter=limiter) for p in probs]
    refs = [oracle_run(p, prec, nsteps=2) for p in probs]
    err = mixed_rel_err if bc == "dirichlet" else max_rel_err
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        dev = lambda a: torch.from_numpy(a).to(DT[prec]).cuda()  # noqa: E731
        items = [dict(shape=p.shape, h=p.h, chi_par=p.chi_par, dt=p.dt, T=dev(p.T0), bx=dev(p.b[0]), by=dev(p.b[1]))
                 for p in probs]
        b = asd.Batch(items, bc=bc, dtype=DT[prec], limiter=limiter)
    for block, body, capacity in ((512, 0, 4), (256, 0, 8), (256, 0, 16), (512, 1, 4), (256, 1, 8), (256, 1, 16)):
        b.set_variant(0)
        b.set_block(block)
        b.set_variant(body)
        b.set_capacity(capacity)
        for mode in (0, 2):
            with torch.cuda.stream(st):
                for p, it in zip(probs, items):
                    it["T"].copy_(dev(p.T0))
                b.step(2, mode)
            st.synchronize()
            for p, it, ref in zip(probs, items, refs):
                assert err(it["T"].double().cpu().numpy(), ref) <= TOL[prec], (block, body, capacity, mode, p.shape)
