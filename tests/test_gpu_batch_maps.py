"""Batches of problems with different sets of material maps (none, sigma,
mu_r, both): each problem runs the code of its own maps under the tiles of
them all.  The bits of the single-problem single-step kernel, in the smallest
and the largest tiles."""
import numpy as np
import pytest

from paper_2405_00814_amd import workloads as W

pytestmark = pytest.mark.gpu

SMALL = [(173, 140), (90, 201), (66, 70), (131, 97)]
LARGE = [(820, 831), (843, 820), (273, 259), (80, 97)]  # enough cells for the largest tiles


@pytest.mark.parametrize("npml", [0, 16])
@pytest.mark.parametrize("shapes", [SMALL, LARGE], ids=["small", "large"])
@pytest.mark.parametrize("maps", [("", "s", "m", "sm"), ("m", "", "m", ""), ("sm", "m", "", "s"), ("sm", "", "sm", "")],
                         ids=["all", "mu", "turned", "both"])
def test_batch_of_mixed_maps(maps, shapes, npml):
    from paper_2405_00814_amd.sim import Batch, Sim
    probs = []
    for q, (shape, m) in enumerate(zip(shapes, maps)):
        rng = np.random.default_rng(q)
        pb = W.dielectric2d(shape[0], ny=shape[1], steps=40, seed=q, nrect=8, side=(8, 30), npml=npml, nprobes=1)
        pb.sigma = rng.uniform(0, 0.02, shape).astype(np.float32) if "s" in m else None
        pb.mu_r = rng.uniform(1, 2, shape).astype(np.float32) if "m" in m else None
        pb.source.cell = (20, 20)
        pb.source.params = (1.0, 6 * pb.dt, 1.0 / (10 * pb.dt))
        pb.probes = np.array([(20, 20), (24, 30), (40, 22)], np.int32)
        probs.append(pb)
    b = Batch(probs)
    for n in (1, 27, 12):
        b.step(n)
    for q, pb in enumerate(probs):
        s = Sim.from_problem(pb)
        s.set_kernel(2)
        s.step(40)
        for f in ("ez", "hx", "hy"):
            got = b.get_field(q, f)
            assert np.abs(got).max() > 0 and np.array_equal(got, s.get_field(f)), (q, f)
        assert np.array_equal(b.probe(q), s.probe()), q
        s.close()
    b.close()
