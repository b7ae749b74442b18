"""GPU: the run lists of brick-stored scales are grouped on the device.  They are
those of the CPU, and building a hierarchy with them takes little longer than
building it without any (with numpy sorting it took half as long again; every
region rebuild pays for it)."""
import time

import numpy as np
import pytest
import torch

from paper_1807_02284_amd import hierarchy, inputs
from paper_1807_02284_amd.level import F32, Level, Params
from test_parity_brick_tiles import surface

pytestmark = pytest.mark.gpu


def tube_scales(nx, ny):
    """Walled box with a brick scale along a tube and a second one inside it."""
    flags = inputs.plume_flags(nx, ny, ny, inlet_radius=6.0, sphere_center=(20.0, ny / 2, ny / 2),
                               sphere_radius=0.0)
    p0 = Params(nu=2e-3, g_max=0.1, tau_s=0.6, u_in=(0.05, 0.0, 0.0), s_in=1.0)
    levels, kinds = [Level(nx, ny, ny, p0, scalar=True, periodic=0, flags=flags)], [flags]
    for k, alpha in enumerate((1.5, 2.0)):
        def tube(px, py, pz, r=0.3 * ny - 10 * k, x0=10 + 18 * k, x1=nx - 20 - 22 * k):
            return (px >= x0) & (px <= x1) & ((py - ny / 2) ** 2 + (pz - ny / 2) ** 2 <= r * r)

        lev, kd = hierarchy.brick_scale([3 + 2 * k] * 3, [nx - 13, ny - 13, ny - 13], alpha, p0, tube,
                                        scalar=True, storage=F32)
        levels.append(lev)
        kinds.append(kd)
    return levels, kinds


@pytest.mark.parametrize("ratio", [2 / 3, 0.75])
def test_device_lists_are_those_of_the_cpu(ratio):
    shape = (88, 72, 64)
    ghosts = surface(shape, (40.3, 35.1, 30.7), 24.0).astype(np.int32)
    cells, offsets = hierarchy.brick_ghost_runs(ghosts, shape, ratio)
    c, o = hierarchy._brick_ghost_runs(torch.as_tensor(ghosts, device="cuda"), shape, ratio)
    np.testing.assert_array_equal(c.cpu().numpy(), cells)
    np.testing.assert_array_equal(o.cpu().numpy(), offsets)
    listed = np.flatnonzero(np.random.default_rng(3).random(88 * 72 * 64) < 0.8).astype(np.int32)
    for bricks in (False, True):
        cells, offsets = hierarchy.brick_post_runs(listed, shape, 1 / ratio, bricks)
        c, o = hierarchy._brick_post_runs(torch.as_tensor(listed, device="cuda"), shape, 1 / ratio, bricks)
        np.testing.assert_array_equal(c.cpu().numpy(), cells)
        np.testing.assert_array_equal(o.cpu().numpy(), offsets)


def test_run_lists_add_little_to_building_a_hierarchy():
    levels, kinds = tube_scales(192, 96)

    def seconds(**kw):
        best = 1e9
        for _ in range(6):
            torch.cuda.synchronize()
            t = time.perf_counter()
            H = hierarchy.Hierarchy(levels, kinds, **kw)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        return best, H

    plain, _ = seconds(tile_posts=False, tile_shells=False)
    tiled, H = seconds()
    assert H.c_scales[1].n_ghost_tiles > 0 and H.c_scales[2].n_post_tiles[1] > 0
    assert tiled <= 1.15 * plain + 2e-3
