"""Staging and flush of a tile's windows at the sizes where they change their
way: axes of the smallest length an order allows, narrower than the windows
(which then hold several periodic images), rows of many widths (a node's place
follows from its number by a reciprocal), and (fewer tiles than groups, then
more) a launch with and without the tile queue.  Against the FP64 oracle."""
import numpy as np
import pytest

import paper_1909_09613_amd as wt
from paper_1909_09613_amd.inputs import RunSpec
from tests import helpers as H

pytestmark = pytest.mark.gpu

PRECISIONS = [wt.PIC_FP64, wt.PIC_MIXED32]
IDS = ["fp64", "fp32"]


@pytest.mark.parametrize("precision", PRECISIONS, ids=IDS)
@pytest.mark.parametrize("ndim,order", [(2, 1), (2, 3), (2, 4), (3, 2), (3, 4)])
def test_smallest_axes(orc, ndim, order, precision):
    spec = RunSpec(ndim, (order + 3,) * ndim, order, 0.45, 20.0, 0.05, 3, 800 + order, colocated=False)
    ex, eu, eE, eB, _ = H.trajectory_vs_oracle(orc, spec, 0.002, 9, precision)
    fp32 = precision == wt.PIC_MIXED32
    assert ex <= (1e-4 if fp32 else 1e-12) and eu <= (1e-4 if fp32 else 1e-12)
    assert max(eE, eB) <= (1e-3 if fp32 else 1e-12)


def _one_step(orc, spec, precision, tile):
    fp32 = precision == wt.PIC_MIXED32
    sp, E, B = H.random_state(spec, 21, 0.05, fp32=fp32)
    g = H.oracle_grid(orc, spec)
    g.E[:] = E
    g.B[:] = B
    g.zero_J()
    ref = H.copy_species(sp)
    for s in ref:
        g.push_species(s["x"], s["u"], s["qm"], s["Q"])
    sim = wt.Sim([spec], precision)
    try:
        wt.pic_set_tiling(sim.ctx, tile)
        sim.set_species(0, sp)
        sim.set_fields(0, E, B)
        sim.gpd()
        got = [sim.particles(0, s) for s in range(2)]
        J = sim.fields(0)[2]
        d = sim.diagnostics(0)
    finally:
        sim.close()
    assert d.n_nonfinite == 0 and d.n_out_of_range == 0
    ex, eu = H.particle_errors(spec, ref, got)
    assert ex <= (2e-6 if fp32 else 1e-12) and eu <= (2e-6 if fp32 else 1e-12)
    scale = H.abs_current_scale(orc, spec, sp, E, B)
    for k in range(3):
        assert np.max(np.abs(J[k] - g.J[k])) / scale[k] <= H.current_tol(spec, k, fp32)


@pytest.mark.parametrize("precision", PRECISIONS, ids=IDS)
@pytest.mark.parametrize("tx", [5, 6, 7, 8, 21, 22, 23, 24, 53, 54, 55, 56])
def test_row_widths_2d(orc, tx, precision):
    # l = 2: after a sort the field rows span tx + 2 or tx + 3 nodes, the
    # current's tx + 4, and one more per side that particles cross
    _one_step(orc, RunSpec(2, (70, 20), 2, 0.45, 50.0, 0.01, 2, 820), precision, (tx, 8, 1))


@pytest.mark.parametrize("precision", PRECISIONS, ids=IDS)
@pytest.mark.parametrize("tile", [(9, 3, 2), (10, 2, 3), (11, 4, 2), (26, 2, 2), (28, 2, 2)])
def test_row_widths_3d(orc, tile, precision):
    _one_step(orc, RunSpec(3, (30, 9, 8), 2, 0.45, 50.0, 0.01, 1, 821), precision, tile)


@pytest.mark.parametrize("precision", PRECISIONS, ids=IDS)
def test_more_tiles_than_groups(orc, precision):
    # 64 x 48 tiles of 4 x 4 cells: more than the groups the chip holds at once
    _one_step(orc, RunSpec(2, (256, 192), 1, 0.45, 50.0, 0.01, 1, 822), precision, (4, 4, 1))


@pytest.mark.parametrize("precision", PRECISIONS, ids=IDS)
@pytest.mark.parametrize("order,tile", [(2, (4, 4, 4)), (3, (8, 4, 4)), (3, (4, 4, 4)), (2, (8, 8, 4)), (2, (8, 3, 4))])
def test_padded_rows_3d(orc, order, tile, precision):
    # rows padded in both windows, in the current's alone and in none (tiles
    # that leave room for one group per CU), and an odd number of rows per plane
    _one_step(orc, RunSpec(3, (18, 13, 11), order, 0.4, 50.0, 0.01, 1, 823), precision, tile)
