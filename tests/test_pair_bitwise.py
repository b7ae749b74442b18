"""GPU: a fused pair of steps (step_pair.hip) is bit for bit two single steps,
so the result of a run depends neither on how it is split into calls nor on
whether its states were stored on the way (cslbm_step_store: single steps,
the recomputation of the differentiable rollout).  Both kernels evaluate one
cell update, so the tolerance is zero."""
import dataclasses

import pytest
import torch

from test_pair_kernels import MARCHING, TILED, WIDE_TILED
from test_parity_pair import level

pytestmark = pytest.mark.gpu

SHAPES = MARCHING + TILED + WIDE_TILED
OPTIONS = [(False, False), (True, True), (True, False), (False, True)]


def state(lev):
    return [t.reshape(-1, lev.plane)[:, : lev.n].clone()
            for t in (lev.f, lev.f_next, lev.g, lev.g_next) if t is not None]


@pytest.mark.parametrize("adaptive", [True, False])
@pytest.mark.parametrize("scalar,force", OPTIONS)
@pytest.mark.parametrize("shape", SHAPES)
def test_one_call_equals_single_step_calls(shape, scalar, force, adaptive):
    n = 9    # four pairs and one step
    lev = level(shape, scalar, force)[0]
    lev.set_params(dataclasses.replace(lev.params, adaptive=adaptive))
    f0, g0 = lev.f.clone(), None if lev.g is None else lev.g.clone()
    lev.step(n)
    got = state(lev)
    lev.f.copy_(f0)
    if scalar:
        lev.g.copy_(g0)
    for _ in range(n):
        lev.step(1)
    for a, b in zip(got, state(lev)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("shape", [(64, 64, 66), (33, 29, 35)])
def test_stored_states_are_those_of_one_call(shape):
    n = 9
    lev = level(shape, True, True)[0]
    f0, g0 = lev.f.clone(), lev.g.clone()
    fs = [torch.zeros_like(f0) for _ in range(n)]
    gs = [torch.zeros_like(g0) for _ in range(n)]
    lev.step_store(f0, g0, fs, gs)
    lev.step(n)
    assert torch.equal(lev.f.reshape(27, -1)[:, : lev.n], fs[-1].reshape(27, -1)[:, : lev.n])
    assert torch.equal(lev.g.reshape(7, -1)[:, : lev.n], gs[-1].reshape(7, -1)[:, : lev.n])
