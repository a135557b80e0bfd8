"""Scratch of the radial spectrum between calls: the column buffer is set up in stream order on the caller's
stream (its first use can follow a call that took the full transform with the same window index), and columns of
a batch that a narrower window does not read hold zeros."""
import math

import numpy as np
import pytest
import torch

from paper_1806_10550_amd import synth
from paper_1806_10550_amd.lib import radial_spectrum, spectrum_release

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_columns_follow_the_full_transform_on_a_side_stream():
    from oracle import radial as R
    n, h0 = 1024, 0.5
    h, ds = synth.random_film(n, 4, 2.0 * math.pi, h0, seed=1)
    qmax = 100.5 * 2.0 * math.pi / (n * ds)
    ref = {s: R.radial_spectrum(h, h0, ds, s, qmax) for s in (1.0, 40.0)}
    s = torch.cuda.Stream()
    spectrum_release()
    with torch.cuda.stream(s):
        ht = torch.from_numpy(h).to(DEV)
        for sigma in (40.0, 1.0, 40.0, 1.0, 1.0):      # 261 columns (full), then 105
            q, v, c = radial_spectrum(ht, ds, h0, sigma, qmax, stream=s)
            qo, vo, co = ref[sigma]
            assert np.array_equal(c, co) and np.max(np.abs(q - qo) / qo) <= 1e-15
            assert np.max(np.abs(v - vo)) <= 1e-12 * np.max(vo) # the spectrum tests' bound


def test_narrow_windows_after_a_wide_one():
    n, h0 = 1024, 0.5
    h, ds = synth.random_film(n, 4, 2.0 * math.pi, h0, seed=2)
    ht = torch.from_numpy(h).to(DEV)
    spectrum_release()
    at = lambda k: radial_spectrum(ht, ds, h0, 0.0, (k + 0.5) * 2.0 * math.pi / (n * ds))
    first = at(70)                                       # 71 columns of a batch of 128
    at(120)
    # each transform of a column left from the wide window would multiply it by up to 32: past the largest double
    # after 205 calls
    for _ in range(230):
        last = at(70)
    assert all(np.array_equal(x, y) for x, y in zip(first, last))


def test_group_scratch_is_sized_by_the_groups():
    """Between a window's inscribed circle and its corners only groups are added: the scratch grows by the added
    groups' means and their index, not by every m between (of which a quarter or fewer are sums of two squares)."""
    n = 4096
    h = torch.full((n, n), 0.5, dtype=torch.float64, device=DEV)
    free = lambda: torch.cuda.mem_get_info()[0]
    spectrum_release()
    k = 2.0 * math.pi / n
    c1 = radial_spectrum(h, 1.0, 0.5, 0.0, (n // 2 + 0.1) * k)[2]
    torch.cuda.empty_cache()
    before = free()
    c2 = radial_spectrum(h, 1.0, 0.5, 0.0, 0.7072 * n * k)[2]
    torch.cuda.empty_cache()
    grown = before - free()
    groups, members = len(c2) - len(c1), int(c2.sum() - c1.sum())
    assert (groups, members) == (338580, 3599105)       # counted on the integers
    # means (8 B) and offsets (4 B) by group, positions (4 B) by member; three allocations of 2 MiB granularity
    assert grown <= 12 * groups + 4 * members + 3 * 2 * (2 << 20)
    spectrum_release()
