"""The hydrostatic correction where a cell's pressure is negative (as a half-step
state's can be): the sound speed of Eqs. (50)-(57) is then no number, and the
dissipation takes the whole jump.  The state itself is refused, but a sweep of
it is finite and the same in FP32 as in FP64.

Bound: the one of the sub-operator tests, max difference over the field's
largest entry 2e-6 (FP32 storage against FP64)."""
import numpy as np
import pytest

import fish_inputs as fi
from oracle import OUTFLOW

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gravity", ["unsplit", "split"])
@pytest.mark.parametrize("d", [0, 1, 2])
def test_sweep_over_a_cell_of_negative_pressure(d, gravity):
    import paper_0910_2854_amd as fish
    n = (12, 11, 10)
    st = fi.sphere_state(n, 7, beta=1.0)
    cell = st["cell"]
    at = (5, 5, 6)
    b = [0.5 * (st["bx"][5, 5, 6] + st["bx"][5, 5, 7]), 0.5 * (st["by"][5, 5, 6] + st["by"][5, 6, 6]),
         0.5 * (st["bz"][5, 5, 6] + st["bz"][6, 5, 6])]
    rest = 0.5 * sum(cell[(k,) + at] ** 2 for k in (1, 2, 3)) / cell[(0,) + at] + 0.5 * sum(x * x for x in b)
    inner = cell[(4,) + at] - rest
    assert inner > 0.0 and min(abs(x) for x in b) > 0.0
    cell[(4,) + at] = rest - 0.3 * inner
    out = []
    for precision in ("fp64", "fp32"):
        g = fish.Box(*n, bc=(OUTFLOW,) * 3, precision=precision, gravity=gravity, hse=True)
        with pytest.raises(fish.FishError):
            g.set_state(st)
        g.sweep("L", d, 0.02 / max(n))
        out.append(g.get_state(check=False)["cell"])
        g.close()
    assert np.all(np.isfinite(out[0]))
    for k in range(5):
        err = np.max(np.abs(out[1][k] - out[0][k])) / np.max(np.abs(out[0]))
        assert err <= 2e-6, (k, err)
