"""The two routes of the radial spectrum (only the columns the window reads, or the whole 2D transform)
against the oracle on both sides of the rule between them, at the edges of the column batches (64,
128) and of the transpose tile, with the window changing from call to call on one film size."""
import math

import numpy as np
import pytest
import torch

from paper_1806_10550_amd import synth
from paper_1806_10550_amd.lib import radial_spectrum

pytestmark = pytest.mark.gpu


def check(h, ds, h0, sigma, qmax):
    from oracle import radial as R
    q, v, c = radial_spectrum(torch.from_numpy(h).to("cuda:0"), ds, h0, sigma, qmax)
    qo, vo, co = R.radial_spectrum(h, h0, ds, sigma, qmax)
    assert len(q) == len(qo) and np.array_equal(c, co)
    assert np.max(np.abs(q - qo) / qo) <= 1e-15
    assert np.max(np.abs(v - vo)) <= 1e-12 * np.max(vo)  # the spectrum tests' bound


# column counts E + 1 (E = floor(sqrt(M)) + ceil(4 sigma)) around the rule 2 (E + 1) <= n/2 + 1
@pytest.mark.parametrize("n,radii", [(16, (1, 2, 3, 4)), (33, (3, 4, 5)), (100, (19, 20, 21, 24, 25, 26)),
                                     (261, (59, 60, 61, 62, 63, 64)), (530, (123, 124, 125, 128, 131, 133))])
@pytest.mark.parametrize("sigma", [0.0, 1.0])
def test_column_routes_match_oracle(n, radii, sigma):
    h, ds = synth.random_film(n, 4, 2.0 * math.pi, 0.5, seed=n)
    for k in radii + radii[:2]:
        check(h, ds, 0.5, sigma, (k + 0.5) * 2.0 * math.pi / (n * ds))
