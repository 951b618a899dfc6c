"""Sweeps of large boxes with streamed accesses (tables above 384 MiB whose rows
are whole 128-byte lines): bitwise the plain sweeps, which the same box takes in
the company of a small one with other rows.  Rows of 255 and 127 cells on outflow
axes, whose last lane holds one cell and whose face row has a whole last pair.

Exact: every cell is computed by the same operations with either access."""
import functools

import numpy as np
import pytest

import fish_inputs as fi
from oracle import OUTFLOW

pytestmark = pytest.mark.gpu
BC = (OUTFLOW,) * 3
SIZES = {"fp32": (255, 157, 165), "fp64": (127, 150, 166)}


@functools.lru_cache(maxsize=1)
def _state(n, gravity):
    if gravity == "none":
        return fi.random_fourier_state(n, seed=2, mach=0.7, beta=3.0, kmax=2)
    return fi.sphere_state(n, 2)


@pytest.mark.parametrize("precision,gravity,hse,limiter", [
    ("fp32", "none", False, "VANLEER"), ("fp32", "none", False, "MINMOD"), ("fp32", "none", False, "MACH_SWITCH"),
    ("fp32", "unsplit", True, "VANLEER"), ("fp32", "split", False, "MINMOD"),
    ("fp64", "none", False, "MINMOD"), ("fp64", "none", False, "VANLEER"), ("fp64", "split", True, "VANLEER")])
def test_streamed_equals_plain(precision, gravity, hse, limiter):
    import paper_0910_2854_amd as fish
    n, esize = SIZES[precision], 4 if precision == "fp32" else 8
    rows = [n[a] + 1 for a in range(3)]
    assert rows[0] * esize % 128 == 0 and 16 * esize * rows[0] * rows[1] * rows[2] > 384 << 20
    print(f"streamed {n} {precision} {gravity} {hse} {limiter}", flush=True)
    st = _state(n, gravity)
    small = fi.uniform_state((5, 4, 3))
    if gravity != "none":
        small["phi"] = np.zeros((3, 4, 5))
    out = []
    for company in (False, True):
        b = fish.Batch(fish.box_pool_bytes(n, precision, gravity != "none", BC) + (1 << 20), precision=precision,
                       gravity=gravity, hse=hse, limiter=getattr(fish, limiter))
        i = b.add(st, bc=BC)
        if company:
            b.add(small)
        b.step(1)
        out.append(b.get(i))
        b.close()
    for k in ("cell", "bx", "by", "bz"):
        assert np.array_equal(out[0][k], out[1][k]), k
    assert out[0]["t"] == out[1]["t"]
