"""GPU: the adjoint of a flagged step clears the padding of its output planes
(elements past the box), also where the grid has fewer threads than there are
padding elements."""
import numpy as np
import pytest
import torch

from paper_1807_02284_amd.level import Level
from test_adjoint_multiscale import flagged_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scalar", [False, True])
@pytest.mark.parametrize("kind", ["walls", "neumann_ghost_odd"])
def test_flagged_adjoint_clears_the_padding(kind, scalar):
    shape, periodic, kinds, p = flagged_case(kind)
    n = int(np.prod(shape))
    lev = Level(*shape, p, scalar=scalar, periodic=periodic, flags=kinds)
    lev.init_equilibrium(np.ones(n), np.zeros((3, n)), np.full(n, 0.5) if scalar else None)

    def planes(q, value):
        return torch.full((q * lev.plane,), value, device="cuda")

    lam1, lam0 = planes(27, 0.0), planes(27, float("nan"))
    mu1, mu0 = (planes(7, 0.0), planes(7, float("nan"))) if scalar else (None, None)
    lam1.reshape(27, -1)[:, :n] = 1e-3
    lev.adjoint_step(lev.f, lev.g, lam1, mu1, lam0, mu0, None)
    for out in (lam0, mu0):
        if out is not None:
            out = out.reshape(-1, lev.plane)
            assert bool((out[:, n:] == 0).all()) and bool(torch.isfinite(out[:, :n]).all())
