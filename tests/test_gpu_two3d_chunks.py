"""The chunk length that the two-step 3D passes choose for the tiles near the
x and y slabs against 16 planes (relative L2 1e-6: the same updates, planes
at a chunk's start recomputed elsewhere) and the oracle (1e-4)."""
import numpy as np
import pytest

from paper_2405_00814_amd import workloads as W

from helpers import rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,npml", [((40, 30, 24), (4,) * 6), ((53, 41, 260), (5, 0, 3, 4, 6, 2)), ((17, 64, 16), (0, 3, 0, 0, 0, 0))])
def test_slab_chunks(shape, npml):
    from oracle import oracle as O
    from paper_2405_00814_amd.sim import Sim
    pb = W.yee3d(shape=shape, steps=20, seed=2, nbox=3, side=(1, 3), npml=0, nprobes=3, tau_steps=3.0)
    pb.npml = npml
    pb.cpml = dict(m=3.0, sigma_max=0.0, kappa_max=3.0, alpha_max=0.05, m_alpha=1.0)
    fields = ("ex", "ey", "ez", "hx", "hy", "hz")
    rng = np.random.default_rng(3)
    init = {f: (rng.standard_normal(shape) * (1 if f[0] == "e" else 1 / 377)).astype(np.float32) for f in fields}
    out = []
    for txo in (0, 16):
        s = Sim.from_problem(pb)
        s.set_kernel(3, (4, 0, 0, txo))
        for f, a in init.items():
            s.set_field(f, a)
        s.step(20)
        out.append({f: s.get_field(f) for f in fields} | {"probe": s.probe()})
        s.close()
    o = O.for_problem(pb)
    o.set_state({f: a.astype(np.float64) for f, a in init.items()})
    rec = o.run(20)
    for f in fields:
        assert rel_l2(out[0][f], getattr(o, f)) <= 1e-4, f
    assert rel_l2(out[0]["probe"], rec) <= 1e-4
    for f in out[0]:
        assert rel_l2(out[0][f], out[1][f]) <= 1e-6, f
