"""The x sweeps' windows of 64 lanes: rows shorter and longer than a window,
odd and even rows (whose last lane holds one cell), rows that end anywhere in
a window, few and many rows per block, both kinds of boundary.

Against the oracle's sub-operator, at the bounds of the other sub-operator
tests: max difference over the field's largest entry 1e-12 (FP64), 2e-6
(FP32 storage against the FP64 oracle)."""
import numpy as np
import pytest

import fish_inputs as fi
from oracle import OUTFLOW, PERIODIC, Oracle

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-12, "fp32": 2e-6}
ROWS = (1, 2, 5, 7, 8, 9, 52, 56, 57, 112, 113, 119, 120, 121, 128, 129, 243)


def max_rel(got, want):
    return max(float(np.max(np.abs(got[k] - want[k])) / (np.max(np.abs(want[k])) + 1e-300))
               for k in ("cell", "bx", "by", "bz"))


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("op", ["L", "B"])
def test_x_sweep_over_row_lengths(op, precision):
    import paper_0910_2854_amd as fish
    for i, nx in enumerate(ROWS):
        n = (nx, 3 + i % 4, 2 + i % 3)
        for bc in ((PERIODIC,) * 3, (OUTFLOW,) * 3, (OUTFLOW, PERIODIC, PERIODIC)):
            st = fi.random_fourier_state(n, seed=40 + i, mach=0.8, beta=2.0, kmax=2)
            o = Oracle(*n, bc=bc)
            o.set_state(st)
            dt = 0.4 / (8.0 * max(n))
            o.apply(op, 0, dt)
            want = o.get_state()
            for target in (None, 64, 700):
                g = fish.Box(*n, bc=bc, precision=precision)
                if target:
                    g.set_shape("fluid_x", target, i % 2)
                    g.set_shape("field_x", target, i % 2)
                g.set_state(st)
                g.sweep(op, 0, dt)
                err = max_rel(g.get_state(check=False), want)
                g.close()
                assert err <= TOL[precision], (n, bc, target, err)
