"""fdtd_last_step_time after an adjoint run: the launches it made, its passes
of several steps counted once."""
import pytest

from paper_2405_00814_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,window", [(100, (50, 100)), (100, (20, 60)), (13, (0, 13))])
def test_launches_of_an_adjoint_run(T, window):
    """All steps kept (no recompute): forward and backward passes, the seed
    of the last step's probes where it is in the window, a gradient each."""
    from paper_2405_00814_amd.sim import Sim
    pb = W.adjoint2d(n=72, steps=T, seed=2, design=(26, 40, 24, 42), npml=8, nprobes=4)
    s = Sim.from_problem(pb)
    TB = s.get_kernel()["tile"][2]
    passes = -(-T // TB)
    s.adjoint_grads(T, window, pb.design, T)
    assert s.last_step_time()[1] == 2 * passes + (window[1] == T) + 2
    s.adjoint_eps(T, window, pb.design, T)
    assert s.last_step_time()[1] == 2 * passes + (window[1] == T) + 1
    s.set_kernel(2)
    s.adjoint_eps(T, window, pb.design, T)
    assert s.last_step_time()[1] == T + passes + (window[1] == T) + 1
    s.close()
