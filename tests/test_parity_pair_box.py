"""GPU: calls of five and more steps on small fully periodic FP32 levels run
pairs of steps on tiles (k_step_pair_box).  Against the FP64 oracle (1e-6 per
step, the one-step tolerance) and against the same number of single-step
calls: two FP32 evaluations of one step differ by at most twice their own
error of 2e-7, per step."""
import numpy as np
import pytest

import oracle
from test_parity_pair import level
from test_parity_single import oparams, rel_err

pytestmark = pytest.mark.gpu

# 8x4x4, 8x6x4 and 16x4x4 tiles: one tile, whole tiles, last tiles of one cell
# in each direction, sides shorter than a tile (single steps), long thin boxes
SHAPES = [(8, 4, 4), (16, 8, 8), (9, 5, 5), (17, 13, 9), (32, 32, 32), (33, 29, 35), (48, 48, 48),
          (57, 55, 58), (15, 121, 41), (160, 9, 13), (7, 20, 20), (20, 3, 20), (20, 20, 3)]


@pytest.mark.parametrize("scalar,force", [(False, False), (True, True), (True, False), (False, True)])
@pytest.mark.parametrize("shape", SHAPES)
def test_tile_pairs_equal_single_steps(shape, scalar, force):
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


@pytest.mark.parametrize("shape,scalar,force", [((9, 5, 5), True, True), ((33, 29, 35), False, False)])
def test_tile_pairs_match_oracle(shape, scalar, force):
    n = 5
    lev, dom, p, f, g = level(shape, scalar, force)
    lev.step(n)
    h, gg = lev.get_populations(shifted=True)
    fo, go = oracle.step(dom, oparams(p), f, g, n_steps=n) if scalar else \
        oracle.step(dom, oparams(p), f, n_steps=n)
    assert rel_err(h.double().cpu().numpy() + oracle.weights()[:, None], fo) <= n * 1e-6
    if scalar:
        np.testing.assert_allclose(gg.double().cpu().numpy(), go, rtol=0, atol=n * 1e-6)
