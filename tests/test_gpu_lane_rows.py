"""y and z sweeps with the lanes along the sweep at the longest rows they take,
which along y depends on the cells along x, and just past them: bitwise the
result of walked segments (a shape that is set).

Exact: every cell is computed by the same operations in either layout."""
import numpy as np
import pytest

import fish_inputs as fi
from oracle import OUTFLOW, PERIODIC
from test_gpu_yz_lanes import MODES, _sweep

pytestmark = pytest.mark.gpu
ROWS = [((1, 712, 5), 1), ((1, 713, 5), 1), ((3, 352, 4), 1), ((3, 353, 4), 1), ((6, 232, 3), 1), ((7, 128, 5), 1),
        ((7, 129, 5), 1), ((6, 5, 128), 2), ((6, 5, 129), 2), ((3, 4, 352), 2)]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("mode", [MODES[0], MODES[3]])
@pytest.mark.parametrize("n,d", ROWS)
def test_lanes_equal_segments(n, d, mode, precision):
    for bc in ((PERIODIC,) * 3, (OUTFLOW,) * 3):
        st = fi.random_fourier_state(n, seed=9, mach=0.7, beta=3.0, kmax=2) if mode[0] == "none" else fi.sphere_state(n, 9)
        for op in "LB":
            got = _sweep(n, bc, st, precision, mode, op, d, None)
            want = _sweep(n, bc, st, precision, mode, op, d, 11)
            for k in ("cell", "bx", "by", "bz"):
                assert np.array_equal(got[k], want[k]), (bc, op, k)
