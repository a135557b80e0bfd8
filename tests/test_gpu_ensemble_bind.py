"""Binding an ensemble's state orders its validation, on the ensemble's own stream, after the work that the caller's
stream still holds."""
import pytest
import torch

from paper_1806_10550_amd.lib import Ensemble

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
NONPOS = 5


def _busy():
    """Some tens of milliseconds of work ahead on the current stream."""
    x = torch.ones(1 << 27, dtype=torch.float64, device=DEV)
    for _ in range(60):
        x.mul_(1.0)


@pytest.mark.parametrize("own", [False, True])
@pytest.mark.parametrize("late", [1.0, -1.0])
def test_state_written_just_before_bind_is_the_one_checked(own, late):
    """A state that turns positive (or negative) by a copy still in the stream's queue at bind."""
    s = torch.cuda.Stream() if own else torch.cuda.current_stream()
    with torch.cuda.stream(s):
        e = Ensemble([64, 96], [80, 48], [0.7, 0.7], [10.0, 10.0], stream=s)
        e.set_scheme(tol=1e-10)
        packed = torch.full((e.size,), -late, dtype=torch.float64, device=DEV)
        src = torch.full_like(packed, late)
        torch.cuda.synchronize()
        _busy()
        packed.copy_(src)
        e.bind(packed)
        status, _, statuses, _ = e.step(1, 0.1)
        torch.cuda.synchronize()
        assert statuses == ([0, 0] if late > 0 else [NONPOS, NONPOS])
        assert status == statuses[0]
        e.close()
