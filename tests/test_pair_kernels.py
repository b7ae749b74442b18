"""Which kernel a call of many steps takes on a fully periodic FP32 level
(step_pair.hip): the small tiles, the march along z or single steps, asked of
the library on the CPU; and each of them against the FP64 oracle at the edges
of its tiles, with scalar and force.  Tolerance: 1e-6 per step, as for one."""
import ctypes as C

import numpy as np
import pytest

import oracle
from paper_1807_02284_amd import _capi
from paper_1807_02284_amd.level import F16S, F32, Params
from test_parity_pair import level
from test_parity_single import oparams, rel_err

SINGLE, TILES, MARCH = 0, 1, 2


def kind(shape, scalar=False, force=False, **kw):
    L = _capi.CslbmLevel()
    L.nx, L.ny, L.nz = shape
    L.storage = kw.get("storage", F32)
    L.periodic = kw.get("periodic", 7)
    L.p = Params(nu=0.01, grad_mode=kw.get("grad_mode", 0)).to_c()
    L.flags = kw.get("flags")   # pointers are looked at for NULL only
    L.g = 0x1000 if scalar else None
    L.force = 0x2000 if force else None
    return getattr(_capi.load(), "_ZN5cslbm14step_pair_kindEPK11cslbm_level")(C.byref(L))


# march, 64-wide tiles: whole ones, a last tile of one column (and a last row
# past a tile), two columns, eight planes; 32-wide: whole, part, shorter rows
MARCHING = [(64, 64, 66), (193, 67, 45), (130, 73, 60), (256, 264, 8), (96, 70, 45), (80, 61, 66), (27, 100, 120)]
# 8x4x4 tiles (too few rows for the others), whole 8x4x4, 8x6x4: last tiles of one
# to three cells in every direction
TILED = [(9, 5, 50), (32, 32, 32), (33, 29, 35), (31, 30, 34), (15, 121, 41), (160, 9, 13)]
WIDE_TILED = [(34, 27, 47), (65, 19, 37)]   # 16x4x4, without the scalar


@pytest.mark.parametrize("scalar,force", [(False, False), (True, True), (True, False), (False, True)])
def test_kernel_of_each_shape(scalar, force):
    for shape in MARCHING:
        assert kind(shape, scalar, force) == MARCH, shape
    for shape in TILED:
        assert kind(shape, scalar, force) == TILES, shape
    for shape in () if scalar else WIDE_TILED:
        assert kind(shape, scalar, force) == TILES, shape
    # sides shorter than a tile; tiles that fill the CUs badly; too few rows
    for shape in [(7, 20, 20), (20, 3, 20), (20, 20, 3), (41, 33, 37), (250, 8, 140), (600, 600, 7)]:
        assert kind(shape, scalar, force) == SINGLE, shape


def test_levels_without_pairs():
    for shape in (MARCHING[0], TILED[0]):
        assert kind(shape, storage=F16S) == SINGLE
        assert kind(shape, periodic=3) == SINGLE
        assert kind(shape, flags=0x3000) == SINGLE
        assert kind(shape, grad_mode=1) == SINGLE
    assert kind((8, 4, 4)) == TILES and kind((8, 4, 4), True) == SINGLE


@pytest.mark.gpu
@pytest.mark.parametrize("shape,scalar,force", [
    ((193, 67, 45), True, True), ((130, 73, 60), True, False), ((256, 264, 8), True, True),
    ((256, 264, 8), False, True), ((193, 67, 45), False, False), ((80, 61, 66), True, True),
    ((96, 70, 45), False, True), ((27, 100, 120), True, True),
    ((9, 5, 50), True, True), ((9, 5, 50), False, False), ((31, 30, 34), True, True), ((33, 29, 35), True, True),
    ((33, 29, 35), False, True), ((15, 121, 41), True, True), ((160, 9, 13), True, False),
    ((34, 27, 47), False, True), ((65, 19, 37), False, False),
])
def test_pairs_match_oracle(shape, scalar, force):
    assert kind(shape, scalar, force) == (MARCH if shape in MARCHING else TILES)
    n = 5
    lev, dom, p, f, g = level(shape, scalar, force)
    lev.step(n)
    h, gg = lev.get_populations(shifted=True)
    fo, go = oracle.step(dom, oparams(p), f, g, n_steps=n) if scalar else \
        oracle.step(dom, oparams(p), f, n_steps=n)
    assert rel_err(h.double().cpu().numpy() + oracle.weights()[:, None], fo) <= n * 1e-6
    if scalar:
        np.testing.assert_allclose(gg.double().cpu().numpy(), go, rtol=0, atol=n * 1e-6)
