"""The adjoint with the interval left open (a longer last segment, as far as
its memory goes) against segments of ceil(sqrt T) steps and one segment:
gradients, loss, record and state are the same bits, for design boxes that
let all steps, some and none beyond the last interval be kept."""
import numpy as np
import pytest
import torch

from paper_2405_00814_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,design,T", [((90, 77), (40, 44, 30, 33), 101), ((90, 77), (20, 60, 20, 56), 101),
                                            ((40, 33), (0, 40, 0, 33), 50), ((300, 41), (150, 250, 10, 30), 37),
                                            ((40, 33), (9, 20, 9, 20), 2)])
def test_open_interval(shape, design, T):
    from paper_2405_00814_amd.sim import Sim
    rng = np.random.default_rng(1)
    dt = 0.6e-3 / 2.99792458e8
    pb = W.Problem(name="adj", ndim=2, shape=shape, dx=(1e-3, 1e-3), dt=dt, steps=T, npml=(6, 0, 5, 4),
                   eps_r=rng.uniform(1, 3, shape).astype(np.float32), sigma=rng.uniform(0, 0.01, shape).astype(np.float32),
                   mu_r=None, source=W.Source((shape[0] // 3, shape[1] // 2), W.SRC_GAUSSIAN, (1.0, 10 * dt, 4 * dt)),
                   probes=np.array([(shape[0] - 9, 12), (12, shape[1] - 9)], np.int32))
    out = []
    for ckpt in (0, int(np.ceil(np.sqrt(T))), T):
        s = Sim.from_problem(pb)
        r = s.adjoint_grads(T, (0, T), design, ckpt)
        got = [np.asarray(x.cpu()) if torch.is_tensor(x) else np.asarray(x) for x in r if x is not None]
        out.append(got + [s.get_field(f) for f in ("ez", "hx", "hy")] + [s.probe()])
        s.step(3)  # the state goes on from T
        out[-1].append(s.get_field("ez"))
        s.close()
    for q in (1, 2):
        assert len(out[0]) == len(out[q])
        for a, b in zip(out[0], out[q]):
            assert np.array_equal(a, b)
