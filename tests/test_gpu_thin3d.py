"""Defaults of 3D grids of few planes: the marching kernel where its
workgroups fill the device and there is no absorbing layer, else one thread
per cell, with the same bits."""
import numpy as np
import pytest

from paper_2405_00814_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,npml,tx", [((3, 816, 816), 0, 16), ((8, 660, 660), 0, 16), ((3, 816, 816), 8, 0),
                                           ((9, 600, 660), 0, 0), ((4, 300, 300), 0, 0), ((3, 816, 814), 0, 0)])
def test_default_of_few_planes(shape, npml, tx):
    from paper_2405_00814_amd.sim import Sim
    rng = np.random.default_rng(1)
    dt = 0.55e-3 / 2.99792458e8
    pb = W.Problem("thin", 3, shape, (1e-3,) * 3, dt, 1, (0, 0) + (npml,) * 4, rng.uniform(1, 4, shape).astype(np.float32), None,
                   None, W.Source(tuple(n // 2 for n in shape), W.SRC_RICKER, (1.0, 8 * dt, 1 / (12 * dt)), component="ez"),
                   np.array([tuple(n // 2 for n in shape)], np.int32))
    init = (rng.standard_normal(shape)).astype(np.float32)
    out = []
    for kernel in (None, (2, (4 if shape[2] % 4 == 0 else 2, 0, 0 if tx else 16))):
        s = Sim.from_problem(pb)
        if kernel is None:
            assert tuple(s.get_kernel()["tile"])[2] == tx and s.get_kernel()["variant"] == 2
        else:
            s.set_kernel(*kernel)
        s.set_field("ez", init)
        s.step(6)
        out.append([s.get_field(f) for f in ("ex", "ey", "ez", "hx", "hy", "hz")] + [s.probe()])
        s.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
