"""Particles through pic_set_particles and pic_get_particles, bit for bit: what
comes back is the input wrapped into the box (and rounded to the FP32 layout in
mixed precision), for positions beyond the box, on its faces, and tiny
negative ones that wrap onto its end; before any step and in several runs.  A
non-finite input is refused and leaves what was loaded as it was."""
import numpy as np
import pytest

import paper_1909_09613_amd as wt
from paper_1909_09613_amd import inputs
from paper_1909_09613_amd.inputs import RunSpec

pytestmark = pytest.mark.gpu


def _expected(spec, x, u, fp32):
    x = x.copy()
    for d in range(spec.ndim):
        n = float(spec.n[d])
        v = np.fmod(x[:, d], n)
        v = np.where(v < 0.0, v + n, v)
        x[:, d] = np.where(v >= n, v - n, v)
    x[:, spec.ndim:] = 0.0
    if fp32:
        x, u = inputs.quantize_fp32(x, u)
        for d in range(spec.ndim):
            x[:, d] = np.where(x[:, d] >= spec.n[d], 0.0, x[:, d])
    return x, u


@pytest.mark.parametrize("precision", [wt.PIC_FP64, wt.PIC_MIXED32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("ndim", [2, 3])
def test_round_trip_and_refusal(ndim, precision):
    fp32 = precision == wt.PIC_MIXED32
    specs = [RunSpec(ndim, n, 1, 0.3, 10.0, 0.1, p, 1) for n, p in (((9, 7, 6)[:ndim], 3), ((31, 8, 5)[:ndim], 1))]
    rng = np.random.default_rng(3)
    sim = wt.Sim(specs, precision)
    try:
        want = {}
        for r, spec in enumerate(specs):
            for s in range(2):
                m = spec.ncell * spec.ppc_s
                x = (rng.random((m, 3)) * 5.0 - 2.0) * np.array(spec.n3)
                x[:8, 0] = [-1e-20, -0.0, 0.0, spec.n[0], -spec.n[0], 3.0, 3.0 - 2.0 ** -30, spec.n[0] - 2.0 ** -30]
                x[8:12, 1] = [-1e-300, 7e15, -7e15, spec.n[1] + 1e-9]
                u = rng.normal(size=(m, 3)) * 3.0
                wt.pic_set_particles(sim.ctx, r, s, x, u)
                want[r, s] = _expected(spec, x, u, fp32)
        for bad in (np.nan, np.inf):
            for which in (0, 1):
                a = [np.full((len(want[0, 0][0]), 3), 1.0), np.full((len(want[0, 0][0]), 3), 1.0)]
                a[which][-1, 1] = bad
                with pytest.raises(wt.PicError) as e:
                    wt.pic_set_particles(sim.ctx, 0, 0, *a)
                assert e.value.status == wt.PIC_ERR_ARG and ("momentum" if which else "position") in str(e.value)
        for (r, s), (x, u) in want.items():
            gx, gu = sim.particles(r, s)
            assert np.array_equal(gx, x) and np.array_equal(gu, u)
    finally:
        sim.close()
