"""GPU: cslbm_vorticity (one pass over the populations, tiles of 64 x 8 cells
walked along z) against central differences in FP64 of the velocity that
cslbm_read_macro returns.  A difference of two FP32 velocities of at most
0.1, each with a few roundings: 2e-7 absolute covers them."""
import numpy as np
import pytest
import torch

from paper_1807_02284_amd import inputs
from paper_1807_02284_amd.level import F16S, F32, Level, Params

pytestmark = pytest.mark.gpu


def curl(u, periodic):
    """|curl u| of u [3][nz][ny][nx]; one-sided at non-periodic faces."""
    g = np.zeros((3, 3) + u.shape[1:])
    for b, axis in enumerate((2, 1, 0)):
        n = u.shape[1 + axis]
        i = np.arange(n)
        lo, hi = (i - 1) % n, (i + 1) % n
        h = np.full(n, 2.0)
        if not periodic & (1 << b):
            lo, hi = np.maximum(i - 1, 0), np.minimum(i + 1, n - 1)
            h = (hi - lo).astype(float)
        for a in range(3):
            d = np.take(u[a], hi, axis) - np.take(u[a], lo, axis)
            shape = [1, 1, 1]
            shape[axis] = n
            hh = h.reshape(shape)
            g[a, b] = np.where(hh > 0, d / np.where(hh > 0, hh, 1.0), 0.0)
    return np.sqrt((g[2, 1] - g[1, 2]) ** 2 + (g[0, 2] - g[2, 0]) ** 2 + (g[1, 0] - g[0, 1]) ** 2)


@pytest.mark.parametrize("shape,periodic,storage,scalar", [
    ((64, 8, 16), 7, F32, False),     # one full tile
    ((65, 9, 5), 7, F32, True),       # one column and row past it
    ((130, 17, 33), 0, F32, False),   # faces on every axis
    ((63, 7, 1), 2, F32, False),      # a single plane
    ((1, 40, 12), 6, F32, True),
    ((1, 3, 2), 0, F32, False),
    ((200, 5, 9), 5, F16S, False),
])
def test_vorticity_against_differences_of_the_velocity(shape, periodic, storage, scalar):
    nx, ny, nz = shape
    n = nx * ny * nz
    flags = None if periodic == 7 else np.zeros(n, np.uint8)
    p = Params(nu=0.01, beta=1e-3 if scalar else 0.0, s_ref=0.1)
    lev = Level(nx, ny, nz, p, storage=storage, scalar=scalar, periodic=periodic, flags=flags)
    u = 0.05 * inputs.perturbation((3, n), 3)
    rho = 1.0 + 0.01 * inputs.perturbation(n, 4)
    s = 0.2 + 0.1 * inputs.perturbation(n, 5) if scalar else None
    lev.init_equilibrium(rho, u, s)
    omega, speed = lev.vorticity()
    _, v, _ = lev.read_macro()
    torch.cuda.synchronize()
    v = v.double().cpu().numpy().reshape(3, nz, ny, nx)
    np.testing.assert_allclose(omega.cpu().numpy(), curl(v, periodic).reshape(-1), rtol=0, atol=2e-7)
    np.testing.assert_allclose(speed.cpu().numpy(), np.sqrt((v ** 2).sum(0)).reshape(-1), rtol=0, atol=2e-7)
