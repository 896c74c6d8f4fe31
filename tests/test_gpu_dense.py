"""Segments of more particles than the sort orders by place within their cells:
in runs where that is a full tile's usual number (more levels in arrival order:
fewer ranks than levels, more, tiles of the fewest cells and of more cells than
are ordered at all) and in a tile that happens to hold more than its share; cells
denser than are ordered.  One step against the FP64 oracle."""
import numpy as np
import pytest

import paper_1909_09613_amd as wt
from paper_1909_09613_amd.inputs import RunSpec
from tests import helpers as H

pytestmark = pytest.mark.gpu

PRECISIONS = [wt.PIC_FP64, wt.PIC_MIXED32]
IDS = ["fp64", "fp32"]
CASES = {
    "levels-hold-all": ((34, 20), 2, 40, (16, 16, 1)),
    "levels-and-more": ((34, 20), 3, 70, (16, 16, 1)),
    "fewest-cells": ((9, 8), 1, 520, (4, 4, 1)),
    "ragged-box": ((9, 6, 7), 2, 140, (4, 4, 4)),
    "box-and-more": ((8, 7, 6), 1, 260, (4, 4, 4)),
    "dense-cells-small-segments": ((17, 12), 2, 70, (8, 8, 1)),
}


@pytest.mark.parametrize("precision", PRECISIONS, ids=IDS)
@pytest.mark.parametrize("name", list(CASES))
def test_dense_runs(orc, name, precision):
    n, order, ppc, tile = CASES[name]
    spec = RunSpec(len(n), n, order, 0.45, 50.0, 0.01, ppc, 840)
    H.check_one_step(orc, spec, precision, tiling=(tile, 3, 2) if len(n) == 2 else (tile, 2, 1))


def test_dense_and_more_cells_than_are_ordered(orc):
    spec = RunSpec(2, (70, 40), 2, 0.45, 50.0, 0.01, 4, 841)
    H.check_one_step(orc, spec, wt.PIC_MIXED32, tiling=((64, 33, 1), 3, 2))


@pytest.mark.parametrize("precision", PRECISIONS, ids=IDS)
def test_one_tile_holds_more_than_its_share(orc, precision):
    # 512 cells of 16 particles a species, and 300 of a neighbour's
    spec = RunSpec(2, (64, 16), 2, 0.45, 50.0, 0.01, 16, 842)

    def place(x):
        rng = np.random.default_rng(5)
        far = np.flatnonzero(x[:, 0] >= 32.0)[:300]
        x[far, :2] = rng.random((300, 2)) * (32.0, 16.0)

    H.check_one_step(orc, spec, precision, tiling=((32, 16, 1), 3, 2), place=place)


def test_runs_of_both_kinds(orc):
    # the dense run holds the fewer particles, and then the more
    for sizes in ((20, 60), (60, 20)):
        specs = [RunSpec(2, (sizes[0], 18), 2, 0.45, 50.0, 0.01, 40, 843),
                 RunSpec(2, (sizes[1] * 8, 17), 2, 0.3, 20.0, 0.01, 4, 844)]
        sim = wt.Sim(specs, wt.PIC_MIXED32)
        try:
            wt.pic_set_tiling(sim.ctx, (16, 16, 1))
            states = [H.random_state(s, 5 + r, 0.05, fp32=True) for r, s in enumerate(specs)]
            for r, (sp, E, B) in enumerate(states):
                sim.set_species(r, sp)
                sim.set_fields(r, E, B)
            sim.gpd()
            for r, (sp, E, B) in enumerate(states):
                g = H.oracle_grid(orc, specs[r])
                g.E[:] = E
                g.B[:] = B
                g.zero_J()
                for s in sp:
                    g.push_species(s["x"], s["u"], s["qm"], s["Q"])
                ex, eu = H.particle_errors(specs[r], sp, [sim.particles(r, s) for s in range(2)])
                assert ex <= 2e-6 and eu <= 2e-6
                d = sim.diagnostics(r)
                assert d.n_nonfinite == 0 and d.n_out_of_range == 0
        finally:
            sim.close()
