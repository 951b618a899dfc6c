"""Sweeps of small tables with one cell per lane: bitwise those of the same box
in a table large enough (more than 1024 rows along every axis) for two, with
rows up to the longest that one window takes (56 cells) and past it.

Exact: every cell is computed by the same operations in either layout."""
import numpy as np
import pytest

import fish_inputs as fi
from oracle import OUTFLOW, PERIODIC

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("gravity,hse", [("none", False), ("split", True)])
@pytest.mark.parametrize("n", [(56, 5, 4), (57, 5, 4), (4, 56, 5), (5, 4, 57), (16, 17, 15)])
def test_one_cell_per_lane_equals_two(n, gravity, hse, precision):
    import paper_0910_2854_amd as fish
    if gravity == "none":
        make = lambda m, seed: fi.random_fourier_state(m, seed=seed, mach=0.7, beta=3.0, kmax=2)
    else:
        make = fi.sphere_state
    for bc in ((PERIODIC,) * 3, (OUTFLOW,) * 3):
        out = []
        for company in (False, True):
            b = fish.Batch(1 << 26, precision=precision, gravity=gravity, hse=hse)
            i = b.add(make(n, 3), bc=bc)
            if company:
                b.add(make((32, 33, 34), 4), bc=bc)
            b.step(2)
            out.append(b.get(i, check=False))
            b.close()
        for k in ("cell", "bx", "by", "bz"):
            assert np.array_equal(out[0][k], out[1][k]), (bc, k)
        assert out[0]["t"] == out[1]["t"]
