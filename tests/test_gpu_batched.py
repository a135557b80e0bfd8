"""Newton iterations enqueued in batches that stand down on the device, against the same films with a test after
every iteration (per-launch timing takes one at a time): every step's record and the state agree bit for bit, with
attempts accepted, exhausted and left inadmissible at different places of a batch."""
import numpy as np
import pytest
import torch

from paper_1806_10550_amd import synth
from paper_1806_10550_amd.lib import Grid

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
DS = synth.CONFIGS["small128"].ds


def run(nx, ny, u, dts, timed, **scheme):
    """Steps from u with the given dt to try (None: the one the control asks for): infos, dt after each, states."""
    g = Grid(nx, ny, DS)
    g.set_model(10.0, 0.1, 3, 2)
    g.set_xsweep("row")
    g.set_scheme(**scheme)
    g.set_diagnostics(True)
    h = torch.from_numpy(u.copy()).to(DEV)
    g.bind(h)
    g.profile(timed)
    out, dt = [], None
    for d in dts:
        st, dt, info = g.try_step(dt if d is None else d)
        torch.cuda.synchronize()
        out.append((st, dt, info, h.cpu().numpy().copy()))
    launches = g.profile_read()["yline"][1]
    g.profile(False)
    g.close()
    return out, launches


ADAPT = dict(tol=1e-10, adaptive=1, dt_min=1e-7, dt_max=4.0, dt_shrink=0.5, dt_grow=1.5, grow_after=2)
SCHEMES = {
    # grown dt: the number of iterations changes from step to step
    "grow": (dict(max_newton=20, **ADAPT), [0.01] + [None] * 14),
    # attempts that run out of iterations inside a batch, or in its last one
    "exhausted": (dict(max_newton=3, **ADAPT), [0.001] + [None] * 6),
    "limit": (dict(max_newton=6, **ADAPT), [2.0, None, 0.05, None, 2.0, None]),
    # iterates that turn negative or not a number at first, then accepted ones
    "inadmissible": (dict(max_newton=12, **ADAPT), [0.1, 3e3, None, 0.1, 4e4, None]),
    # fixed dt: a step that fails leaves the state as it was
    "fixed": (dict(tol=1e-10, max_newton=12, adaptive=0), [0.001, 500.0, 0.001, 0.002]),
    "trapezoidal": (dict(theta=0.5, max_newton=9, **ADAPT), [0.5] + [None] * 5),
}


@pytest.mark.parametrize("nx,ny", [(128, 128), (61, 300), (1100, 40), (40, 1100)])
@pytest.mark.parametrize("name", SCHEMES)
def test_batches_agree_with_single_iterations(nx, ny, name):
    scheme, dts = SCHEMES[name]
    u = synth.noise_film(nx, ny, seed=nx + ny, amp=0.2)
    single, launches = run(nx, ny, u, dts, True, **scheme)
    batched, none = run(nx, ny, u, dts, False, **scheme)
    assert none == 0                                        # (not timed: batches)
    assert launches == sum(x[2]["total_iters"] for x in single)
    for s, b in zip(single, batched):
        assert s[:3] == b[:3]
        assert np.array_equal(s[3], b[3])
    if name == "inadmissible":
        assert any(x[2]["rejections"] for x in single)
    if name == "fixed":
        assert any(x[0] != 0 for x in single) and any(x[0] == 0 for x in single)
