"""Upload and download of a box: what is set is what is got, in the storage
precision, with face n of a periodic axis equal to face 0.  Boxes that go in
one piece on one thread, in one piece on several, and in chunks through the
two staging buffers (more than 32 MB); boundaries of either kind.

Exact: the values are only copied and converted."""
import numpy as np
import pytest

from oracle import OUTFLOW, PERIODIC

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("bc", [(PERIODIC,) * 3, (OUTFLOW,) * 3, (PERIODIC, OUTFLOW, PERIODIC)])
@pytest.mark.parametrize("n", [(3, 2, 2), (9, 1, 7), (40, 33, 21), (96, 80, 64), (170, 150, 160)])
def test_round_trip(n, bc, precision):
    import paper_0910_2854_amd as fish
    nx, ny, nz = n
    rng = np.random.default_rng(nx)
    st = {"cell": rng.uniform(0.5, 1.0, (5, nz, ny, nx)), "bx": rng.uniform(-0.1, 0.1, (nz, ny, nx + 1)),
          "by": rng.uniform(-0.1, 0.1, (nz, ny + 1, nx)), "bz": rng.uniform(-0.1, 0.1, (nz + 1, ny, nx))}
    st["cell"][4] += 3.0  # positive pressure
    g = fish.Box(*n, bc=bc, precision=precision)
    for turn in range(2):  # the staging buffers in either turn
        st["cell"][0] += 0.25
        g.set_state(st)
        out = g.get_state()
        for k in ("cell", "bx", "by", "bz"):
            want = st[k].astype(np.float32).astype(np.float64) if precision == "fp32" else st[k].copy()
            if k != "cell":
                a = "xyz".index(k[1])
                if bc[a] == PERIODIC:
                    f = np.moveaxis(want, 2 - a, 0)
                    f[-1] = f[0]
            assert np.array_equal(out[k], want), (k, turn)
    g.close()
