"""A particle's place in its tile's windows and its cell after the move: tiles
that touch the grid's periodic ends and tiles that do not, axes narrower than a
tile's windows (whose box is then centred in the axis), and particles that
leave their stencil upwards, downwards or stay, in the same wave.  Some steps
from identical state against the FP64 oracle; the boxes drift across the ends
meanwhile.  Tolerances: those of the multi-step comparisons at this length
(FP64 rounding, and FP32 rounding of the state over ten steps)."""
import numpy as np
import pytest

import paper_1909_09613_amd as wt
from paper_1909_09613_amd.inputs import RunSpec
from tests import helpers as H

pytestmark = pytest.mark.gpu

GRIDS = {
    "2d-inner-and-ends": ((48, 40), 2, (8, 8, 1)),
    "2d-cubic": ((64, 33), 3, (16, 8, 1)),
    "2d-x-narrow": ((7, 40), 2, (4, 8, 1)),
    "2d-y-narrow": ((40, 6), 3, (16, 4, 1)),
    "3d": ((18, 13, 16), 2, (4, 4, 4)),
    "3d-z-narrow": ((18, 16, 6), 2, (4, 4, 4)),
}


@pytest.mark.parametrize("precision", [wt.PIC_FP64, wt.PIC_MIXED32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("beam", ["up", "down", "both"])
@pytest.mark.parametrize("grid", list(GRIDS), ids=list(GRIDS))
def test_places_and_moves(orc, grid, beam, precision):
    n, order, tile = GRIDS[grid]
    fp32 = precision == wt.PIC_MIXED32
    spec = RunSpec(len(n), n, order, 0.4, 20.0, 0.05, 2 if len(n) == 2 else 1, 900, colocated=False)
    sp, E, B = H.random_state(spec, 31, 0.002, fp32=fp32)
    for s in sp:
        if beam == "down":
            s["u"][:] = -s["u"]
        elif beam == "both":
            s["u"][::2] = -s["u"][::2]
    g = H.oracle_grid(orc, spec)
    g.E[:] = E
    g.B[:] = B
    ref = H.copy_species(sp)
    sim = wt.Sim([spec], precision)
    try:
        wt.pic_set_tiling(sim.ctx, tile)
        sim.set_species(0, sp)
        sim.set_fields(0, E, B)
        sim.step(10)
        d = sim.diagnostics(0)
        got = [sim.particles(0, s) for s in range(2)]
        Eg, Bg, _ = sim.fields(0)
    finally:
        sim.close()
    for _ in range(10):
        g.step(ref)
    assert d.n_nonfinite == 0 and d.n_out_of_range == 0
    ex, eu = H.particle_errors(spec, ref, got)
    assert ex <= (1e-4 if fp32 else 1e-12) and eu <= (1e-4 if fp32 else 1e-12)
    tol = 1e-3 if fp32 else 1e-12
    assert max(H.rel_maxnorm(Eg, g.E)) <= tol and max(H.rel_maxnorm(Bg, g.B)) <= tol
