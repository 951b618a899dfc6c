"""The autotuner on boxes so small that the planned shape, which no set one
equals, is by far the fastest (32^3 FP32: a y sweep of 7 us on lanes along it, of
11 us or more on segments): it is what stays, and results do not change."""
import numpy as np
import pytest

import fish_inputs as fi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(24, 24, 24), (32, 32, 32), (16, 30, 40)])
def test_planned_shapes_stay(n):
    import paper_0910_2854_amd as fish
    st = fi.random_fourier_state(n, seed=6, mach=0.6, beta=3.0, kmax=2)
    out = []
    for tune in (False, True):
        g = fish.Box(*n, precision="fp32")
        g.set_state(st)
        if tune:
            chosen = g.autotune(reps=10)
            for kind in ("fluid_y", "fluid_z", "field_y", "field_z"):
                assert chosen[kind]["target"] == 64 and chosen[kind]["alt_layout"] == 0, chosen
        g.strang_step(0.0)
        out.append(g.get_state())
        g.close()
    for k in ("cell", "bx", "by", "bz"):
        assert np.array_equal(out[0][k], out[1][k])
