"""The CFL reduction across the waves of a block (combined in LDS, published
by the last wave): the fastest cell wherever it sits, boxes of one wave up to
a ragged last block, and blocks that hold several boxes of a batch.

Oracle: the FP64 CPU oracle's CFL step, on the same state.  Tolerance 1e-12 relative
in FP64 (the square roots' and reciprocals' last ulps; the maximum itself is
exact), and 1e-6 in FP32 (speeds in the storage precision)."""
import numpy as np
import pytest

import fish_inputs as fi
from oracle import Oracle

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-12, "fp32": 1e-6}


def spiked_state(n, cell, vmax):
    """A uniform box at rest, but for one cell moving at vmax along x."""
    st = fi.uniform_state(n, rho=1.0, p=0.6, b=(0.3, 0.2, 0.1))
    i, j, k = cell
    st["cell"][1, k, j, i] = vmax
    st["cell"][4, k, j, i] += 0.5 * vmax * vmax
    return st


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [(5, 3, 2), (64, 1, 1), (40, 13, 5), (70, 9, 11), (33, 40, 17)])
@pytest.mark.parametrize("where", ["first", "middle", "last"])
def test_fastest_cell_of_a_box(n, where, precision):
    import paper_0910_2854_amd as fish
    cell = {"first": (0, 0, 0), "middle": tuple(m // 2 for m in n), "last": tuple(m - 1 for m in n)}[where]
    st = spiked_state(n, cell, 2.5)
    o = Oracle(*n)
    o.set_state(st)
    g = fish.Box(*n, precision=precision)
    g.set_state(st)
    tol = TOL[precision]
    assert abs(g.cfl_dt() / o.cfl_dt() - 1.0) <= tol  # the check kernel
    # the reduction fused into the last sweep of a step that hardly moves the
    # state (twelve sub-operators of dt speed / h <= 3e-12 each)
    g.strang_step(1e-14)
    assert abs(g.cfl_dt() / o.cfl_dt() - 1.0) <= tol + 1e-10
    g.close()


def test_blocks_of_several_boxes():
    import paper_0910_2854_amd as fish
    rng = np.random.default_rng(4)
    shapes = [tuple(int(v) for v in rng.integers(2, 9, 3)) for _ in range(23)] + [(40, 20, 10), (3, 3, 3)]
    speeds = rng.uniform(0.5, 4.0, len(shapes))
    batch = fish.Batch(sum(fish.box_pool_bytes(n, "fp64") for n in shapes) + 4096, precision="fp64")
    want = []
    for n, v in zip(shapes, speeds):
        st = spiked_state(n, tuple(int(rng.integers(0, m)) for m in n), float(v))
        o = Oracle(*n)
        o.set_state(st)
        want.append(o.cfl_dt())
        batch.add(st)
    batch.step(1)
    for i, dt in enumerate(want):  # t advanced by two sub-steps of the box's own CFL step
        assert abs(batch.info(i)["t"] / (2.0 * dt) - 1.0) <= 1e-12, (i, shapes[i])
    batch.close()
