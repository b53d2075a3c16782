"""fdtd_step_profile on 2D grids in workgroup tiles: its entry is a pass as
fdtd_step would run it, also of fewer steps than a pass may take, and the
state advances as by fdtd_step."""
import numpy as np
import pytest

from paper_2405_00814_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps,per", [(2, 2), (8, 8), (12, 12), (20, 10), (25, 9), (1, 1)])
def test_profile_of_a_pass(steps, per):
    from paper_2405_00814_amd.sim import Sim
    pb = W.dielectric2d(200, ny=170, steps=40, seed=2, nrect=3, side=(6, 20), npml=8, nprobes=2)
    a, b = Sim.from_problem(pb), Sim.from_problem(pb)
    for s in (a, b):
        s.set_kernel(3, (64, 0, 12))
        s.step(5)
    p = a.step_profile(steps)
    b.step(steps)
    assert len(p) == 1 and p[0]["steps"] == per and p[0]["launches"] == 1 and p[0]["ms"] > 0
    assert a.steps_done() == b.steps_done()
    for f in ("ez", "hx", "hy"):
        assert np.array_equal(a.get_field(f), b.get_field(f))
    assert np.array_equal(a.probe(), b.probe())
    a.close()
    b.close()
