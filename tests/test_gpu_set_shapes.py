"""Set shapes other than the defaults, which stand for the planned ones: bitwise
the result of the planned shapes (of small boxes, lanes along the y and z sweeps),
with and without the alternative layouts."""
import numpy as np
import pytest

import fish_inputs as fi
from test_gpu_shapes import BOXES, FIELDS, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("box", BOXES, ids=lambda b: "x".join(map(str, b[0])))
def test_set_shapes_give_the_planned_result_bitwise(prec, box):
    n, bc, seed = box
    st = fi.random_fourier_state(n, seed=seed, mach=0.7, beta=3.0, kmax=2)
    ref = _run(n, bc, st, prec, None)
    for v in ((400, 63, 0, 1), (385, 65, 1, 0), (1536, 64, 1, 1)):
        got = _run(n, bc, st, prec, v)
        for k in FIELDS:
            assert np.array_equal(got[k], ref[k]), (v, k)
