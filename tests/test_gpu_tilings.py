"""Explicit tilings whose windows need more than half a CU's LDS, and nearly all of
it: 3D mixed precision near the limit (where rows of the particle kernel's fixed
pitches would exceed it and bare rows do not) and beside it, both windows at
the fixed pitches, one of them too wide for its pitch, and a 2D tile of more cells
than the sort orders by place.  One step against the FP64 oracle."""
import pytest

import paper_1909_09613_amd as wt
from paper_1909_09613_amd.inputs import RunSpec
from tests import helpers as H

pytestmark = pytest.mark.gpu

TILES_3D = [(3, (15, 4, 11)), (3, (8, 4, 4)), (2, (19, 2, 15)), (2, (16, 4, 14)), (2, (16, 4, 15)), (2, (16, 4, 12)),
            (2, (18, 4, 4)), (1, (19, 3, 6)), (1, (20, 2, 4))]


@pytest.mark.parametrize("order,tile", TILES_3D)
def test_large_windows_3d(orc, order, tile):
    spec = RunSpec(3, (40, 9, 31), order, 0.45, 50.0, 0.01, 1, 830)
    H.check_one_step(orc, spec, wt.PIC_MIXED32, tiling=(tile, 2, 1))


def test_more_cells_than_are_ordered_2d(orc):
    spec = RunSpec(2, (130, 70), 2, 0.45, 50.0, 0.01, 2, 831)
    H.check_one_step(orc, spec, wt.PIC_MIXED32, tiling=((64, 33, 1), 3, 2))
