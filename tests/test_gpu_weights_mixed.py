"""The closed forms of the interpolation weights in mixed precision, per order and
over the Courant numbers where T_l changes its form: a small time step, one
near c dt = dx / 2, exactly there (T_l = W_l) and just above it (l + 2 nodes, the
tables).  One step from identical state against the FP64 oracle, to the one-step
bounds of mixed precision."""
import pytest

import paper_1909_09613_amd as wt
from paper_1909_09613_amd.inputs import RunSpec
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ndim", [2, 3])
@pytest.mark.parametrize("order", [1, 2, 3, 4])
@pytest.mark.parametrize("a", [0.02, 0.31, 0.499999, 0.5, 0.500001])
def test_weights_over_courant(orc, ndim, order, a):
    n = (24, 18) if ndim == 2 else (12, 10, 9)
    spec = RunSpec(ndim, n, order, a, 20.0, 0.05, 4 if ndim == 2 else 1, 710, colocated=False)
    H.check_one_step(orc, spec, wt.PIC_MIXED32, amp=0.3, seed=9)
