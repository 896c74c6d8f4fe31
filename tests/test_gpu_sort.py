"""The sort's count and scatter passes at the sizes where they can go wrong:
fewer particles than one thread block takes at once, one block's share of 2048
exactly and one cell's particles more, several runs whose ends fall inside a
wave, and particles spread so that neighbouring lanes hold different tiles.  A
sort of a shuffled store must keep every particle: positions and momenta come
back in identity order as one step of the FP64 oracle leaves them."""
import numpy as np
import pytest

import paper_1909_09613_amd as wt
from paper_1909_09613_amd.inputs import RunSpec
from tests import helpers as H

pytestmark = pytest.mark.gpu

CASES = {
    "one-wave": [RunSpec(2, (6, 5), 2, 0.45, 50.0, 0.01, 1, 901)],
    "one-block": [RunSpec(2, (32, 32), 2, 0.45, 50.0, 0.01, 1, 902)],
    "one-block-and-a-row": [RunSpec(2, (32, 33), 2, 0.45, 50.0, 0.01, 1, 903)],
    "runs-within-waves": [RunSpec(2, (7, 5 + k), 2, 0.3, 20.0, 0.01, 1 + k % 2, 910 + k) for k in range(9)],
    "box": [RunSpec(3, (17, 9, 11), 1, 0.45, 50.0, 0.01, 2, 904)],
}


@pytest.mark.parametrize("precision", [wt.PIC_FP64, wt.PIC_MIXED32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("name", list(CASES))
def test_sort_keeps_every_particle(orc, name, precision):
    specs = CASES[name]
    fp32 = precision == wt.PIC_MIXED32
    states = []
    sim = wt.Sim(specs, precision)
    try:
        for r, spec in enumerate(specs):
            sp, E, B = H.random_state(spec, 31 + r, 0.05, fp32=fp32)
            rng = np.random.default_rng(r)
            for s in sp:  # a store in no order at all
                o = rng.permutation(len(s["x"]))
                s["x"], s["u"] = s["x"][o], s["u"][o]
            states.append((sp, E, B))
            sim.set_species(r, sp)
            sim.set_fields(r, E, B)
        sim.gpd()
        for r, spec in enumerate(specs):
            sp, E, B = states[r]
            g = H.oracle_grid(orc, spec)
            g.E[:] = E
            g.B[:] = B
            g.zero_J()
            ref = H.copy_species(sp)
            for s in ref:
                g.push_species(s["x"], s["u"], s["qm"], s["Q"])
            ex, eu = H.particle_errors(spec, ref, [sim.particles(r, s) for s in range(2)])
            assert ex <= (2e-6 if fp32 else 1e-12) and eu <= (2e-6 if fp32 else 1e-12)
            d = sim.diagnostics(r)
            assert d.n_nonfinite == 0 and d.n_out_of_range == 0 and d.n_sorts == 1
    finally:
        sim.close()
