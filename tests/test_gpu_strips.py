"""D(u) on both sides of the line between strips of four and of sixteen rows (2^23 cells), with ragged last strips,
against the oracle."""
import numpy as np
import pytest
import torch

from paper_1806_10550_amd import synth
from paper_1806_10550_amd.lib import Grid

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("nx,ny", [(131, 64035), (131, 64037), (64039, 131)])
@pytest.mark.parametrize("model", ["power", "nlc"])
def test_flux_divergence_of_large_films(orc, model, nx, ny):
    assert (nx * ny > 1 << 23) == ((nx, ny) != (131, 64035))
    h0, ds = {"power": (1.0, 0.67), "nlc": (0.5, 0.13)}[model]
    u = synth.noise_film(nx, ny, seed=nx, h0=h0, amp=0.1 * h0)
    g = Grid(nx, ny, ds)
    if model == "power":
        g.set_model(10.0, 0.1, 3, 2)
        M = orc.Model(kappa=10.0, b=0.1, n=3.0, m=2.0)
    else:
        g.set_model_nlc()
        M = orc.Model.nlc()
    ug = torch.from_numpy(u).to(DEV)
    out = g.flux_divergence(ug, torch.empty_like(ug))
    # the parity tests' bound for this operator: 1e-12 of the largest value
    ref = orc.flux_divergence(M, u, ds)
    assert np.max(np.abs(out.cpu().numpy() - ref)) <= 1e-12 * np.max(np.abs(ref))
    g.close()


def test_theta_half_ensemble_on_both_strip_lengths():
    """b^n of films on both sides of the line in one ensemble: the single films' results, bit for bit."""
    from paper_1806_10550_amd.lib import Ensemble
    nx, ny, ds, dt = [131, 131, 40], [64037, 64035, 51], 0.67, 0.02
    scheme = dict(theta=0.5, tol=1e-10, max_newton=40)
    e = Ensemble(nx, ny, [ds] * 3, [10.0] * 3)
    e.set_scheme(**scheme)
    packed = torch.empty(e.size, dtype=torch.float64, device=DEV)
    films = [torch.from_numpy(synth.noise_film(a, b, seed=b, amp=0.01)).to(DEV) for a, b in zip(nx, ny)]
    for f, u in enumerate(films):
        e.view(packed, f).copy_(u)
    e.bind(packed)
    assert e.step(1, dt)[0] == 0
    for f, u in enumerate(films):
        g = Grid(nx[f], ny[f], ds)
        g.set_model(10.0, 0.1, 3, 2)
        g.set_scheme(**scheme)
        g.bind(u)
        g.step(dt)
        torch.cuda.synchronize()
        assert torch.equal(u, e.view(packed, f)), f
        g.close()
    e.close()
