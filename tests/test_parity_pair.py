"""GPU: calls of five and more steps on fully periodic FP32 levels run fused
pairs of steps (step_pair.hip).  Against the FP64 oracle (1e-6 per step, the
one-step tolerance) and against the same number of single-step calls, which
take the general kernel: two FP32 evaluations of one step differ by at most
twice their own error of 2e-7, per step."""
import numpy as np
import pytest

import oracle
from paper_1807_02284_amd import inputs
from paper_1807_02284_amd.level import Level, Params
from test_parity_single import odomain, oparams, perturbed_start, rel_err, start_fields

pytestmark = pytest.mark.gpu

# 64-wide tiles: full, one column and row past a tile, last tiles of a few
# cells, eight planes; 32-wide: half-line rows, rows shorter than a tile
SHAPES = [(64, 64, 66), (129, 67, 41), (121, 61, 50), (200, 170, 8), (250, 8, 140),
          (96, 70, 45), (80, 61, 66), (27, 100, 120)]


def level(shape, scalar, force):
    nx, ny, nz = shape
    p = Params(nu=0.01, g_max=0.05, tau_s=0.6, beta=1e-3 if scalar else 0.0, s_ref=0.1)
    rho, u = start_fields(nx, ny, nz, 5)
    noise = 1e-4 * inputs.perturbation((27, nx * ny * nz), 6)
    rng = np.random.default_rng(7)
    theta = 1e-4 * rng.standard_normal((3, rho.size)) if force else None
    s = rng.uniform(0.0, 0.3, rho.size) if scalar else None
    lev = Level(nx, ny, nz, p, scalar=scalar, force=theta)
    dom = odomain(nx, ny, nz, theta=theta)
    f, g = perturbed_start(lev, dom, rho, u, noise, s)
    return lev, dom, p, f, g


@pytest.mark.parametrize("scalar,force", [(False, False), (True, True), (True, False), (False, True)])
@pytest.mark.parametrize("shape", SHAPES)
def test_pairs_equal_single_steps(shape, scalar, force):
    n = 6 if scalar else 9    # 2 pairs and 2 steps; 4 pairs and 1 step
    lev, _, _, _, _ = level(shape, scalar, force)
    f0, g0 = lev.f.clone(), None if lev.g is None else lev.g.clone()
    lev.step(n)
    got = [t.clone() for t in (lev.f, lev.f_next, lev.g, lev.g_next) if t is not None]
    lev.f.copy_(f0)
    if g0 is not None:
        lev.g.copy_(g0)
    for _ in range(n):
        lev.step(1)
    ref = [t for t in (lev.f, lev.f_next, lev.g, lev.g_next) if t is not None]
    w = oracle.weights()
    for k, (a, b) in enumerate(zip(got, ref)):
        q = 27 if k < 2 else 7
        a = a.double().cpu().numpy().reshape(q, -1)[:, : lev.n]
        b = b.double().cpu().numpy().reshape(q, -1)[:, : lev.n]
        shift = w[:, None] if q == 27 else 0.0
        scale = np.maximum(np.abs(b + shift), w[:, None] if q == 27 else 0.05)
        assert np.max(np.abs(a - b) / scale) <= n * 4e-7


@pytest.mark.parametrize("shape,scalar,force", [((129, 67, 41), True, True), ((96, 70, 45), False, False)])
def test_pairs_match_oracle(shape, scalar, force):
    n = 5
    lev, dom, p, f, g = level(shape, scalar, force)
    lev.step(n)
    h, gg = lev.get_populations(shifted=True)
    fo, go = oracle.step(dom, oparams(p), f, g, n_steps=n) if scalar else \
        oracle.step(dom, oparams(p), f, n_steps=n)
    assert rel_err(h.double().cpu().numpy() + oracle.weights()[:, None], fo) <= n * 1e-6
    if scalar:
        np.testing.assert_allclose(gg.double().cpu().numpy(), go, rtol=0, atol=n * 1e-6)


def test_calls_of_four_steps_are_four_single_steps():
    lev, _, _, _, _ = level((64, 64, 66), False, False)
    f0 = lev.f.clone()
    lev.step(4)
    a = lev.f.clone()
    lev.f.copy_(f0)
    for _ in range(4):
        lev.step(1)
    assert bool((a == lev.f).all())
