"""fdtd_get_field of the explicit graph, which gathers small grids on the host
and others on the device: host and device results agree bit for bit with the
field that was set, on both sides of the line, with and without the split
field (whose Ez is the sum of two nodes)."""
import numpy as np
import pytest

from paper_2405_00814_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("split", [0, 1])
@pytest.mark.parametrize("shape", [(20, 31), (128, 128), (128, 129), (150, 133)])
def test_fields(shape, split):
    import torch
    from paper_2405_00814_amd.sim import Sim
    pb = W.dielectric2d(shape[0], ny=shape[1], steps=4, seed=2, nrect=2, side=(3, 6), npml=4, nprobes=1)
    pb.sigma = None
    pb.cpml = dict(m=3.0, sigma_max=0.0, kappa_max=1.0, alpha_max=0.0, m_alpha=1.0, split=split)
    s = Sim.from_problem(pb, graph=True)
    rng = np.random.default_rng(1)
    for f in ("ez", "hx", "hy"):
        a = rng.standard_normal(shape).astype(np.float32)
        s.set_field(f, a)
        assert np.array_equal(s.get_field(f), a), f
    s.step(3)
    for f in ("ez", "hx", "hy"):
        d = torch.empty(shape, device="cuda")
        s.get_field_device(f, d)
        assert np.array_equal(s.get_field(f), d.cpu().numpy()), f
    s.close()
