"""GPU: cslbm_vorticity on boxes of every shape: narrow ones and thin axes
walked along z with tiles of their own width, flat ones and binary16 boxes of
short rows in two passes.  Against central differences in FP64 of the velocity
that cslbm_read_macro returns, with the tolerance of test_parity_vorticity; and
no shape takes many times the read-back of its velocity (2 x 600 x 600 cells took
many of them with tiles of 64 columns)."""
import numpy as np
import pytest
import torch

from paper_1807_02284_amd import inputs
from paper_1807_02284_amd.level import F16S, F32, Level, Params
from test_parity_vorticity import curl

pytestmark = pytest.mark.gpu


def level(shape, periodic, storage, scalar, force):
    nx, ny, nz = shape
    n = nx * ny * nz
    flags = None if periodic == 7 else np.zeros(n, np.uint8)
    p = Params(nu=0.01, beta=1e-3 if scalar else 0.0, s_ref=0.1)
    theta = 1e-4 * inputs.perturbation((3, n), 9) if force else None
    lev = Level(nx, ny, nz, p, storage=storage, scalar=scalar, periodic=periodic, flags=flags, force=theta)
    u = 0.05 * inputs.perturbation((3, n), 3)
    rho = 1.0 + 0.01 * inputs.perturbation(n, 4)
    s = 0.2 + 0.1 * inputs.perturbation(n, 5) if scalar else None
    lev.init_equilibrium(rho, u, s)
    return lev


@pytest.mark.parametrize("shape,periodic,storage,scalar,force", [
    ((1, 130, 110), 7, F32, False, False),     # walked: one column, wrapped and not
    ((1, 130, 110), 0, F32, True, True),
    ((2, 100, 130), 6, F32, False, True),
    ((7, 131, 100), 1, F32, True, False),
    ((33, 61, 70), 0, F16S, False, True),      # one tile of 33 columns
    ((80, 70, 50), 7, F32, True, True),        # two of 40
    ((129, 1, 600), 5, F32, False, False),     # 43 columns, a single row
    ((129, 9, 130), 0, F32, False, True),
    ((300, 301, 2), 3, F32, True, False),      # two planes
    ((1030, 1024, 1), 0, F32, False, True),    # two passes: flat
    ((1024, 1030, 1), 7, F32, True, False),
    ((5, 200, 100), 2, F16S, True, True),      # two passes: short rows
    ((31, 60, 70), 7, F16S, False, False),
])
def test_vorticity_of_narrow_and_flat_boxes(shape, periodic, storage, scalar, force):
    nx, ny, nz = shape
    lev = level(shape, periodic, storage, scalar, force)
    omega, speed = lev.vorticity()
    _, v, _ = lev.read_macro()
    torch.cuda.synchronize()
    v = v.double().cpu().numpy().reshape(3, nz, ny, nx)
    np.testing.assert_allclose(omega.cpu().numpy(), curl(v, periodic).reshape(-1), rtol=0, atol=2e-7)
    np.testing.assert_allclose(speed.cpu().numpy(), np.sqrt((v ** 2).sum(0)).reshape(-1), rtol=0, atol=2e-7)


def microseconds(call):
    best = 1e9
    for _ in range(6):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(20):
            call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 50)
    return best


@pytest.mark.parametrize("shape,storage", [((2, 600, 600), F32), ((1, 512, 512), F32), ((8, 400, 400), F16S),
                                           ((16, 256, 256), F32), ((1024, 1024, 1), F32)])
def test_vorticity_takes_a_few_read_backs(shape, storage):
    lev = level(shape, 7, storage, False, False)
    assert microseconds(lev.vorticity) <= 3.0 * microseconds(lev.read_macro) + 20.0
