"""The sort's arrange pass at the sizes where it changes its way: segments of
exactly as many particles as it orders by place within their cells (16 per
cell in a tile of 512 cells), of one particle per cell more (ranked in arrival
order), and cells of just as many particles as it ranks by their keys, one
more and many more.  One step from identical state against the FP64 oracle,
and the particles' identities after it, to the one-step tolerances."""
import numpy as np
import pytest

import paper_1909_09613_amd as wt
from paper_1909_09613_amd import inputs
from paper_1909_09613_amd.inputs import RunSpec
from tests import helpers as H

pytestmark = pytest.mark.gpu

CASES = {
    # spec, tile, particles per species gathered into single cells
    "one-segment-full": (RunSpec(2, (32, 16), 3, 0.45, 50.0, 0.01, 16, 601), (32, 16, 1), ()),
    "one-segment-over": (RunSpec(2, (32, 16), 3, 0.45, 50.0, 0.01, 17, 602), (32, 16, 1), ()),
    "dense-cells-2d": (RunSpec(2, (40, 24), 2, 0.45, 50.0, 0.01, 4, 603), (16, 16, 1), (64, 65, 300)),
    "dense-cells-3d": (RunSpec(3, (20, 12, 10), 2, 0.45, 50.0, 0.01, 2, 604), (8, 4, 4), (64, 65, 300)),
    "cubic-3d": (RunSpec(3, (19, 12, 10), 3, 0.35, 50.0, 0.01, 2, 605), (4, 4, 4), (64, 65)),
}


@pytest.mark.parametrize("precision", [wt.PIC_FP64, wt.PIC_MIXED32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("name", list(CASES))
def test_one_step_arranged(orc, name, precision):
    spec, tile, dense = CASES[name]
    fp32 = precision == wt.PIC_MIXED32
    sp, E, B = H.random_state(spec, 7, 0.05, fp32=fp32)
    rng = np.random.default_rng(8)
    for s in sp:
        p = 0
        for k, m in enumerate(dense):
            for d in range(spec.ndim):
                s["x"][p:p + m, d] = 3 + 2 * k + rng.random(m)
            p += m
        if fp32:
            s["x"], s["u"] = inputs.quantize_fp32(s["x"], s["u"])
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


# one segment per species of a thread's first item and one less or more, and of
# whole batches of items and a remainder, up to more than the pass orders
SEGMENTS = [(31, 11, 3), (32, 16, 2), (41, 5, 5), (31, 11, 6), (41, 5, 10), (45, 7, 13), (32, 16, 8), (41, 5, 20),
            (45, 13, 14), (41, 10, 20)]


@pytest.mark.parametrize("precision", [wt.PIC_FP64, wt.PIC_MIXED32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("nx,ny,ppc", SEGMENTS, ids=["%d" % (a * b * c) for a, b, c in SEGMENTS])
def test_segment_sizes(orc, nx, ny, ppc, precision):
    spec = RunSpec(2, (nx, ny), 2, 0.45, 50.0, 0.01, ppc, 610)
    fp32 = precision == wt.PIC_MIXED32
    sp, E, B = H.random_state(spec, 9, 0.05, fp32=fp32)
    g = H.oracle_grid(orc, spec)
    g.E[:] = E
    g.B[:] = B
    g.zero_J()
    ref = H.copy_species(sp)
    for s in ref:
        g.push_species(s["x"], s["u"], s["qm"], s["Q"])
    sim = wt.Sim([spec], precision)
    try:
        wt.pic_set_tiling(sim.ctx, (nx, ny, 1))
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
