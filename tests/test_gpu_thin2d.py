"""2D grids of few long rows: short calls run single steps, longer ones tiles
of 32 rows, with the same bits; and no length of call takes longer than the
single-step kernel by more than a fifth (they took 2.6 times as long)."""
import numpy as np
import pytest

from paper_2405_00814_amd import workloads as W

pytestmark = pytest.mark.gpu


def _problem(nx, ny):
    rng = np.random.default_rng(2)
    dt = 0.6e-3 / 2.99792458e8
    return W.Problem(name="thin", ndim=2, shape=(nx, ny), dx=(1e-3, 1e-3), dt=dt, steps=1, npml=(0, 0, 8, 8),
                     eps_r=rng.uniform(1, 4, (nx, ny)).astype(np.float32), sigma=None, mu_r=None,
                     source=W.Source((nx // 2, ny // 2), W.SRC_RICKER, (1.0, 6 * dt, 1.0 / (10 * dt))),
                     probes=np.array([(nx // 2, ny // 2 + 2), (nx - 1, ny // 2 - 3)], np.int32))


@pytest.mark.parametrize("nx,ny", [(3, 200000), (8, 100000), (12, 90001), (31, 40000)])
def test_short_and_long_calls(nx, ny):
    from paper_2405_00814_amd.sim import Sim
    pb = _problem(nx, ny)
    a, b = Sim.from_problem(pb), Sim.from_problem(pb)
    assert a.get_kernel()["tile"][:2] == (64, 0)
    b.set_kernel(2)
    for n in (2, 3, 5, 8, 30):
        ta = tb = 1e9
        for _ in range(5):
            a.step(n)
            b.step(n)
            ta, tb = min(ta, a.last_step_time()[0]), min(tb, b.last_step_time()[0])
        assert ta < 1.2 * tb, (n, ta, tb)
    for f in ("ez", "hx", "hy"):
        assert np.array_equal(a.get_field(f), b.get_field(f)), f
    assert np.array_equal(a.probe(), b.probe())
    if nx == 3:  # two single steps, not one pass
        a.step(2)
        assert a.last_step_time()[1] == 2
    a.close()
    b.close()
