"""The y and z fluid sweeps in FP64 with the limiter switch or an irregular
mesh: bitwise the same with the loads one position ahead (a launch of at most
1024 waves) as without, at odd and even positions per segment.

Exact: every cell is computed by the same operations in either loop."""
import numpy as np
import pytest

import fish_inputs as fi
from oracle import OUTFLOW, PERIODIC

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("limiter,stretch", [("MACH_SWITCH", 0.0), ("VANLEER", 0.3), ("MACH_SWITCH", 0.3)])
@pytest.mark.parametrize("bc", [(PERIODIC,) * 3, (OUTFLOW,) * 3])
def test_ahead_or_not(bc, limiter, stretch):
    import paper_0910_2854_amd as fish
    n = (200, 36, 40)  # 125 and 113 waves of rows: segments of 3 cells are above the line
    st = fi.random_fourier_state(n, seed=3, mach=0.7, beta=3.0, kmax=2)
    for d in (1, 2):
        out = []
        for target in (40, 17, 8, 3):
            g = fish.Box(*n, bc=bc, precision="fp64", limiter=getattr(fish, limiter))
            if stretch:
                for a in range(3):
                    w = 1.0 + stretch * np.sin(2.0 * np.pi * (np.arange(n[a]) + 0.5) / n[a])
                    g.set_spacing(a, w / w.sum())
            g.set_shape("fluid_" + "xyz"[d], target)
            g.set_state(st)
            g.sweep("L", d, 0.05 / max(n))
            out.append(g.get_state(check=False))
            g.close()
        for got in out[:-1]:
            assert np.array_equal(got["cell"], out[-1]["cell"]), (d, bc)
