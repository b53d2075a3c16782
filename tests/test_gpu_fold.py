"""The coefficients folded on the device are those of the same formulas in
NumPy's float64, rounded once: one step from Ez alone on a grid without
layers shows Ca and Cb of every cell, a step from Hx shows Db (bitwise, from
values of one)."""
import numpy as np
import pytest

from paper_2405_00814_amd import workloads as W

pytestmark = pytest.mark.gpu
EPS0, MU0 = 8.8541878128e-12, 1.25663706212e-6


@pytest.mark.parametrize("n", [3, 33, 257])
@pytest.mark.parametrize("maps", ["", "e", "s", "es", "m", "esm"])
def test_fold(n, maps):
    from paper_2405_00814_amd.sim import Sim
    rng = np.random.default_rng(n)
    shape = (n, n + 2)
    dt = 0.6e-3 / 2.99792458e8
    m = {k: (rng.uniform(lo, hi, shape).astype(np.float32) if k in maps else None)
         for k, lo, hi in (("e", 1, 12), ("s", 0, 3), ("m", 1, 5))}
    s = Sim(shape, (1e-3, 1e-3), dt, m["e"], m["m"], m["s"], (0,) * 4)
    e = EPS0 * (np.ones(shape) if m["e"] is None else m["e"].astype(np.float64))
    h = (0.0 if m["s"] is None else m["s"].astype(np.float64)) * dt / (2.0 * e)
    ca = ((1.0 - h) / (1.0 + h)).astype(np.float32) * np.ones(shape, np.float32)
    # uniform Ez of one: H stays 0 inside (differences are 0), Ez' = Ca Ez
    one = np.ones(shape, np.float32)
    s.set_field("ez", one)
    s.set_kernel(1)
    s.step(1)
    got = s.get_field("ez")
    inner = (slice(2, n - 1), slice(2, n + 1))
    assert np.array_equal(got[inner], ca[inner])
    s.close()
    # a checkerboard of Ez far below its H leaves Hy' = Db (Ez(i+1) - Ez(i)) / dx
    s = Sim(shape, (1.0, 1.0), dt, m["e"], m["m"], m["s"], (0,) * 4)
    ez = (np.indices(shape)[0] % 2).astype(np.float32)
    s.set_field("ez", ez)
    s.set_kernel(1)
    s.step(1)
    db = (dt / (MU0 * (np.ones(shape) if m["m"] is None else m["m"].astype(np.float64)))).astype(np.float32)
    want = db[:-1] * (ez[1:] - ez[:-1])
    assert np.array_equal(s.get_field("hy")[:-1], want)
    # and Ez' = Ca Ez + Cb ((Hy - Hy(i-1)) / dx), rounded in FP32
    # (but for the last column, next to which Hx is not 0)
    cb = ((dt / e) / (1.0 + h)).astype(np.float32)
    hy = s.get_field("hy").astype(np.float64)
    a, b = (slice(1, None), slice(1, -1)), (slice(0, -1), slice(1, -1))
    ref = ca[a].astype(np.float64) * ez[a] + cb[a].astype(np.float64) * (hy[a] - hy[b])
    assert np.abs(s.get_field("ez")[a] - ref).max() <= 4 * 2.0 ** -24 * max(1.0, np.abs(ref).max())
    s.close()
