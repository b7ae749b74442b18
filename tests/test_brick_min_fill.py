"""GPU: a caller's tile_min_fill holds for the post lists of brick-stored scales
too: no run lists when none can be full enough, run lists for every list at 0,
and the default asks for BRICK_TILE_MIN_FILL entries."""
import pytest

from paper_1807_02284_amd import hierarchy
from paper_1807_02284_amd.level import F32
from test_parity_brick_tiles import build

pytestmark = pytest.mark.gpu


def tiles(**kw):
    H = build(F32, False, (1.5, 2.0), False, **kw)
    return {(i, j): (H.c_scales[i].n_post_tiles[j], H.c_scales[i].n_post[j]) for i, j in H.post}


def test_tile_min_fill_of_brick_lists():
    every, default, none = tiles(tile_min_fill=0), tiles(), tiles(tile_min_fill=10 ** 6)
    coincide = {k for k, (t, _) in every.items() if t == 0}   # mapped from nodes, never in tiles
    assert set(every) - coincide
    for k, (t, n) in every.items():
        assert none[k][0] == 0
        if k not in coincide:
            assert default[k][0] == (t if n >= hierarchy.BRICK_TILE_MIN_FILL * t else 0)
