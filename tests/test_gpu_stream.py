"""The row-streaming kernels (D(u) and J_D^T mu: a wave marches down a strip of columns) against the
oracle at the edges of their strips: owned columns (60 and 58), rows per wave (16 and 8) and per
workgroup (64 and 32), one below, at and above each, and the smallest films; every model."""
import numpy as np
import pytest
import torch

from paper_1806_10550_amd import synth
from paper_1806_10550_amd.lib import Grid

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SHAPES = [(4, 4), (5, 7), (58, 8), (59, 9), (60, 16), (61, 17), (116, 31), (117, 32), (120, 33), (121, 63), (63, 64),
          (64, 65), (57, 130)]


@pytest.mark.parametrize("nx,ny", SHAPES)
@pytest.mark.parametrize("model", ["power", "nlc", "polymer", "linear"])
def test_flux_divergence_and_transposed_jacobian(orc, model, nx, ny):
    h0, ds = {"power": (1.0, 0.67), "nlc": (0.5, 0.13), "polymer": (3.9, 0.13), "linear": (1.0, 0.5)}[model]
    u = synth.noise_film(nx, ny, seed=nx * 100 + ny, h0=h0, amp=0.1 * h0)
    mu = np.random.default_rng(nx + ny).standard_normal((ny, nx))
    g = Grid(nx, ny, ds)
    if model == "power":
        g.set_model(10.0, 0.1, 3, 2)
        M = orc.Model(kappa=10.0, b=0.1, n=3.0, m=2.0)
    else:
        getattr(g, "set_model_" + model)()
        M = orc.Model.linear(1.0, 1.0) if model == "linear" else getattr(orc.Model, model)()
    ug, mg = torch.from_numpy(u).to(DEV), torch.from_numpy(mu).to(DEV)
    out = torch.empty_like(ug)
    # the parity tests' bound for these operators: 1e-12 of the largest value
    ref = orc.flux_divergence(M, u, ds)
    g.flux_divergence(ug, out)
    assert np.max(np.abs(out.cpu().numpy() - ref)) <= 1e-12 * np.max(np.abs(ref))
    ref = orc.jacobian_apply_t(M, u, mu, ds)
    g.jacobian_apply_t(ug, mg, out)
    assert np.max(np.abs(out.cpu().numpy() - ref)) <= 1e-12 * np.max(np.abs(ref))
    g.close()
