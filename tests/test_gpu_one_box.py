"""A table of one box, whose sweeps take it without a look-up: bitwise the same
box in a table of three, from any slot, after steps and after the others leave.

Exact: every cell is computed by the same operations for either table."""
import numpy as np
import pytest

import fish_inputs as fi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [(5, 4, 4), (33, 17, 9), (64, 50, 40)])
@pytest.mark.parametrize("keep", [0, 2])
def test_one_of_three(keep, n, precision):
    import paper_0910_2854_amd as fish
    states = [fi.random_fourier_state(n, seed=s, mach=0.7, beta=3.0, kmax=2) for s in range(3)]
    out = []
    for others_leave_first in (True, False):
        b = fish.Batch(1 << 27, precision=precision)
        ids = [b.add(st) for st in states]
        for part in (0, 1):
            if part == (0 if others_leave_first else 1):
                for k in range(3):
                    if k != keep:
                        b.remove(ids[k])
            b.step(2)
        out.append(b.get(ids[keep]))
        b.close()
    for k in ("cell", "bx", "by", "bz"):
        assert np.array_equal(out[0][k], out[1][k]), k
    assert out[0]["t"] == out[1]["t"]
