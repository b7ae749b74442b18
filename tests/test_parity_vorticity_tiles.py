"""GPU: both kernels of cslbm_vorticity against central differences in FP64 of
the velocity that cslbm_read_macro returns: boxes of up to 768 tiles of
16 x 4 x 4 cells are read tile by tile (8x4x4, 16x6x4 or 16x4x4), larger ones
are walked along z.  The tolerance is that of test_parity_vorticity."""
import pytest

import test_parity_vorticity as vorticity
from paper_1807_02284_amd.level import F16S, F32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,periodic,storage,scalar", [
    ((8, 4, 4), 7, F32, False),       # one tile of 8x4x4
    ((9, 5, 5), 3, F32, True),        # one cell past it on every axis
    ((48, 48, 40), 7, F16S, False),   # 16x6x4
    ((47, 43, 41), 0, F32, True),     # 16x6x4, part tiles and faces
    ((97, 20, 50), 5, F32, False),    # 16x4x4, part tiles
    ((192, 16, 64), 7, F32, False),   # the last size of the tiles: 768
    ((193, 16, 64), 7, F32, True),    # the first that is walked
    ((130, 70, 41), 0, F32, False),   # walked, faces on every axis
    ((65, 129, 33), 2, F16S, True),
])
def test_vorticity_of_small_and_large_boxes(shape, periodic, storage, scalar):
    vorticity.test_vorticity_against_differences_of_the_velocity(shape, periodic, storage, scalar)
