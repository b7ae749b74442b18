"""Exchanges of brick-stored scales through LDS: the run lists partition the
cell lists (CPU), and a hierarchy that uses them computes bitwise the states
of one that gathers every exchange directly (GPU)."""
import numpy as np
import pytest

from paper_1807_02284_amd import hierarchy, inputs
from paper_1807_02284_amd.level import F16S, F32, Level, Params

gpu = pytest.mark.gpu


def surface(shape, centre, radius):
    """Ghost cells (box indices) of the bricks that hold a ball."""
    nx, ny, nz = shape
    z, y, x = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    ball = (x - centre[0]) ** 2 + (y - centre[1]) ** 2 + (z - centre[2]) ** 2 <= radius ** 2
    _, kinds = hierarchy.brick_kinds(ball)
    return np.flatnonzero(kinds == hierarchy.GHOST)


@pytest.mark.parametrize("ratio", [2 / 3, 3 / 4, 0.5, 1.0])
def test_ghost_runs_partition_the_surface_and_fit_the_buffer(ratio):
    shape = (48, 40, 56)
    ghosts = surface(shape, (22.3, 19.1, 30.7), 13.0)
    cells, offsets = hierarchy.brick_ghost_runs(ghosts, shape, ratio)
    np.testing.assert_array_equal(np.sort(cells), np.sort(ghosts))
    assert offsets[0] == 0 and offsets[-1] == cells.size
    assert np.all(np.diff(offsets) > 0) and np.all(np.diff(offsets) <= hierarchy.POST_RUN)
    for a, b in zip(offsets[:-1], offsets[1:]):
        run = cells[a:b].astype(np.int64)
        xyz = (run % 48, (run // 48) % 40, run // (48 * 40))
        box = np.prod([np.floor(np.ptp(v) * ratio) + 2 for v in xyz])
        assert box <= hierarchy.SHELL_TILE_BUFFER


@pytest.mark.parametrize("dst_bricks", [False, True])
@pytest.mark.parametrize("ratio", [4 / 3, 1.5, 2.0, 3.0])
def test_post_runs_partition_the_list_and_fit_the_buffer(dst_bricks, ratio):
    rng = np.random.default_rng(3)
    cells = np.flatnonzero(rng.random(40 * 24 * 16) < 0.8)
    out, offsets = hierarchy.brick_post_runs(cells, (40, 24), ratio, dst_bricks)
    np.testing.assert_array_equal(np.sort(out), cells)
    assert offsets[0] == 0 and offsets[-1] == out.size and np.all(np.diff(offsets) <= hierarchy.POST_RUN)
    for a, b in zip(offsets[:-1], offsets[1:]):
        run = out[a:b].astype(np.int64)
        xyz = (run % 40, (run // 40) % 24, run // (40 * 24))
        assert np.prod([np.floor(np.ptp(v) * ratio) + 2 for v in xyz]) <= hierarchy.POST_TILE_BUFFER


def build(storage, scalar, alphas, dense_last, **kw):
    """Walled reference box with a tube-shaped brick scale and a second scale
    inside it (a smaller tube in bricks, or a dense box)."""
    nx, ny, nz = 80, 56, 48
    flags = inputs.plume_flags(nx, ny, nz, inlet_radius=6.0, sphere_center=(20.0, 28.0, 24.0),
                               sphere_radius=0.0)
    p0 = Params(nu=2e-3, g_max=0.1, tau_s=0.6, u_in=(0.05, 0.0, 0.0), s_in=1.0)
    lev0 = Level(nx, ny, nz, p0, storage=storage, scalar=scalar, periodic=0, flags=flags)
    u = 0.03 * inputs.perturbation((3, lev0.n), 4) * (flags == 0)
    s = 0.5 + 0.4 * inputs.perturbation(lev0.n, 5) if scalar else None
    lev0.init_equilibrium(None, u, s)

    def tube(x0, x1, r):
        return lambda px, py, pz: (px >= x0) & (px <= x1) & ((py - 28.3) ** 2 + (pz - 24.1) ** 2 <= r * r)

    levels, kinds = [lev0], [flags]
    a1, k1 = hierarchy.brick_scale((3, 3, 3), (74, 50, 42), alphas[0], p0, tube(10, 60, 13.0),
                                   scalar=scalar, storage=storage)
    levels.append(a1)
    kinds.append(k1)
    if dense_last:
        a2, k2 = hierarchy.fine_scale((24, 23, 19), (42, 33, 29), alphas[1], p0, scalar=scalar,
                                      storage=storage)
    else:
        a2, k2 = hierarchy.brick_scale((20, 20, 16), (46, 36, 32), alphas[1], p0, tube(28, 38, 3.0),
                                       scalar=scalar, storage=storage)
    levels.append(a2)
    kinds.append(k2)
    for a, b in zip(levels[:-1], levels[1:]):
        hierarchy.fill_from_parent(a, b)
    return hierarchy.Hierarchy(levels, kinds, **kw)


@gpu
@pytest.mark.parametrize("storage,scalar,alphas,dense_last", [
    (F32, True, (1.5, 2.0), False),
    (F32, False, (4 / 3, 2.0), False),
    (F16S, True, (1.5, 2.0), True),
    (F32, True, (1.5, 2.25), True),
])
def test_tiled_brick_exchanges_are_bitwise_the_direct_gather(storage, scalar, alphas, dense_last):
    tiled = build(storage, scalar, alphas, dense_last)
    plain = build(storage, scalar, alphas, dense_last, tile_posts=False, tile_shells=False)
    assert all(tiled.c_scales[i].n_ghost_tiles > 0 for i in (1, 2))
    assert any(tiled.c_scales[i].n_post_tiles[j] > 0 for i in (1, 2) for j in range(i))
    assert all(plain.c_scales[i].n_ghost_tiles == 0 for i in (1, 2))
    for H in (tiled, plain):
        H.step(3)
    for a, b in zip(tiled.levels, plain.levels):
        assert a.count_nonfinite() == 0
        assert bool((a.f == b.f).all())
        if scalar:
            assert bool((a.g == b.g).all())
