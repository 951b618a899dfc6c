"""The van Leer limiter's products over the range of FP32: flux differences of
1.1e19, whose doubled product (2.4e38) is a number and whose fourfold one is not.

Against the oracle, at the bound of the sub-operator tests: max difference over
the field's largest entry 2e-6 (FP32 storage against the FP64 oracle)."""
import numpy as np
import pytest

import fish_inputs as fi
from oracle import OUTFLOW, Oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("limiter", ["VANLEER", "MACH_SWITCH"])
@pytest.mark.parametrize("target", [None, 11])
@pytest.mark.parametrize("d", [0, 1, 2])
def test_sweep_of_a_steep_ramp(d, target, limiter):
    import paper_0910_2854_amd as fish
    n = [5, 6, 4]
    n[d] = 24
    st = fi.uniform_state(tuple(n), p=1.0)
    # a pressure ramp at rest: the energy's flux differences are +-(c/2) dE
    shape = [1, 1, 1]
    shape[2 - d] = 24
    p = (1.0 + 0.05 * np.arange(24.0))
    c = np.sqrt(5.0 / 3.0 * np.maximum(p[1:], p[:-1]))
    diff = 0.5 * c * np.diff(1.5 * p)
    scale = 1.1e19 / np.sqrt(np.max(diff[1:] * diff[:-1]))
    st["cell"][0] = scale
    st["cell"][4] = scale * 1.5 * np.broadcast_to(p.reshape(shape), st["cell"][4].shape)
    o = Oracle(*n, bc=(OUTFLOW,) * 3, limiter=getattr(fish, limiter))
    o.set_state(st)
    dt = 1e-3 / 24
    o.apply("L", d, dt)
    want = o.get_state()["cell"]
    g = fish.Box(*n, bc=(OUTFLOW,) * 3, precision="fp32", limiter=getattr(fish, limiter))
    if target:
        g.set_shape("fluid_" + "xyz"[d], target)
    g.set_state(st)
    g.sweep("L", d, dt)
    got = g.get_state()["cell"]
    g.close()
    assert np.max(np.abs(got - want)) <= 2e-6 * np.max(np.abs(want))
