"""The per-step mass record where iterations are not batched (partitioned sweeps, per-launch timing): the records
of the x sweep are combined once per accepted step, however many iterations and rejected attempts it took, and
the result is that of the accepted state."""
import math

import numpy as np
import pytest
import torch

from paper_1806_10550_amd import synth
from paper_1806_10550_amd.lib import Grid

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# whole lines (timed), partitioned rows, partitioned columns, both
@pytest.mark.parametrize("nx,ny,xsweep", [(130, 70, "row"), (130, 70, "partitioned"), (40, 2100, "row"),
                                          (70, 2100, "partitioned")])
def test_records_are_combined_once_per_accepted_step(nx, ny, xsweep):
    g = Grid(nx, ny, synth.CONFIGS["small128"].ds)
    g.set_model(10.0, 0.1, 3, 2)
    g.set_xsweep(xsweep)
    g.set_scheme(theta=1.0, tol=1e-10, max_newton=5, adaptive=1, dt_min=1e-6, dt_max=1.0, dt_shrink=0.5, dt_grow=1.1,
                 grow_after=5)
    g.set_diagnostics(True)
    h = torch.from_numpy(synth.noise_film(nx, ny, seed=nx, amp=0.05)).to(DEV)
    g.bind(h)
    g.profile(True)
    dt, rejections, iterations = 1.0, 0, 0
    for s in range(6):
        res = g.step(dt)
        dt = res.dt_next
        rejections += res.info["rejections"]
        iterations += res.info["total_iters"]
        torch.cuda.synchronize()
        a = h.cpu().numpy()
        exact = math.fsum(a.ravel())
        # the mass tests' bound: a compensated sum in a fixed order
        assert abs(res.info["mass"] - exact) <= 4 * np.finfo(float).eps * abs(exact)
        assert res.info["hmin"] == float(np.min(a))
    launches = g.profile_read()["mass"][1]
    g.profile(False)
    g.close()
    assert rejections > 0 and iterations > 12
    assert launches == 6 + 1 # (one more checks the bound state before the first step)
