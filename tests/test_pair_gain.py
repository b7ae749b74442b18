"""GPU: a call of many steps on a small box is not slower per step than calls of
four, which take single steps.  Boxes whose tiles fill their last round over
the CUs, and one of few rows, where pairs of steps once took up to 28 % longer."""
import pytest
import torch

from test_parity_pair import level

pytestmark = pytest.mark.gpu


def microseconds(lev, calls, steps):
    best = 1e9
    for _ in range(8):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(calls):
            lev.step(steps)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / (calls * steps))
    return best


@pytest.mark.parametrize("shape,force", [((98, 16, 43), True), ((86, 140, 14), True), ((41, 99, 17), True),
                                         ((52, 30, 49), False), ((83, 15, 56), False),
                                         ((96, 28, 141), True)])
def test_long_calls_are_not_slower_per_step(shape, force):
    lev = level(shape, False, force)[0]
    assert microseconds(lev, 3, 80) <= 1.06 * microseconds(lev, 60, 4)
