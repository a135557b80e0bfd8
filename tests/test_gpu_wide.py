"""Films with very many short lines: on both sides of the lines between the whole-line kernels and the tile passes
(columns of one and up to three tiles, rows of one tile) the sweep taken and the iterate against the oracle."""
import numpy as np
import pytest
import torch

from paper_1806_10550_amd import synth
from paper_1806_10550_amd.lib import Grid, xsweep_choice

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def iterate(orc, nx, ny):
    """Kernels used and error of one iterate over its update (the parity tests' measure)."""
    ds, dt = 0.67347, 0.2
    un = synth.noise_film(nx, ny, seed=nx + ny, amp=0.01)
    g = Grid(nx, ny, ds)
    g.set_model(10.0, 0.1, 3, 2)
    a = torch.from_numpy(un).to(DEV)
    out = torch.empty_like(a)
    g.profile(True)
    e, r, flags = g.newton_iteration(a, a, out, dt)
    used = {k for k, v in g.profile_read().items() if v[1]}
    g.profile(False)
    g.close()
    ref, e_ref, r_ref = orc.adi_iteration(orc.Model(kappa=10.0, b=0.1, n=3.0, m=2.0), un, un, ds, dt, 1.0)
    assert flags == 0 and e == pytest.approx(e_ref, rel=1e-8) and r == pytest.approx(r_ref, rel=1e-9)
    assert np.max(np.abs(out.cpu().numpy() - ref)) <= 1e-10 * np.max(np.abs(ref - un)) + 1e-15
    return used


@pytest.mark.parametrize("nx,ny,whole", [(12288, 4, True), (12289, 4, False), (12288, 64, True), (12289, 64, False),
                                         (16384, 65, True), (16385, 65, False), (16385, 192, False), (16385, 193, True)])
def test_short_columns(orc, nx, ny, whole):
    used = iterate(orc, nx, ny)
    assert ("yline" in used) == whole and ("relations_y" in used) != whole


@pytest.mark.parametrize("nx,ny,whole", [(64, 20480, True), (64, 20481, False), (5, 20481, False), (65, 20481, True)])
def test_short_rows(orc, nx, ny, whole):
    assert xsweep_choice(nx, ny) == ("row" if whole else "partitioned")
    used = iterate(orc, nx, ny)
    assert ("xrow" in used) == whole and ("relations_x" in used) != whole
