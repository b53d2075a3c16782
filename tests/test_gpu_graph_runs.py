"""GPU parity of the explicit graph's layers laid out as runs of rows: sizes
at the edges of a run (64 rows), ragged layers, uniform and varying weights,
sources inside and in the layers, probes there and on the walls, against the
oracle (relative L2 1e-4) and the implicit stepper (1e-5: the same update
summed in another order); short rows and long runs take both layouts."""
import numpy as np
import pytest

from paper_2405_00814_amd import workloads as W

from helpers import rel_l2

pytestmark = pytest.mark.gpu
FIELDS = ("ez", "hx", "hy")


@pytest.mark.parametrize("mat", [0, 1, 2, 3])
@pytest.mark.parametrize("shape,npml,src", [((9, 7), (0,) * 4, ((4, 3), (5, 4))), ((65, 33), (0,) * 4, ((1, 1), (65, 2))),
                                            ((66, 40), (0,) * 4, ((1, 5), (66, 6))), ((130, 41), (8, 0, 5, 7), ((3, 2), (120, 3))),
                                            ((201, 97), (12,) * 4, ((100, 40), (101, 80)))])
def test_graph_runs(shape, npml, src, mat):
    from oracle import oracle as O
    from paper_2405_00814_amd.sim import Sim
    rng = np.random.default_rng(5)
    dt = 0.6e-3 / 2.99792458e8
    field = lambda lo, hi, on: rng.uniform(lo, hi, shape).astype(np.float32) if on else None
    pb = W.Problem(name="graph", ndim=2, shape=shape, dx=(1e-3, 1e-3), dt=dt, steps=40, npml=npml,
                   eps_r=field(1, 4, mat), sigma=field(0, 0.01, mat >= 2), mu_r=field(1, 2, mat == 3),
                   source=W.Source(src[0], W.SRC_RICKER, (1.0, 8 * dt, 1.0 / (12 * dt)), hi=src[1]),
                   probes=np.zeros((0, 2), np.int32),
                   cpml=dict(m=3.0, sigma_max=0.0, kappa_max=3.0, alpha_max=0.05, m_alpha=1.0))
    cells = [(1, 1), tuple(n - 1 for n in shape), tuple(n // 2 for n in shape), (shape[0] // 2, shape[1] // 2)]
    init = {f: (rng.standard_normal(shape) * (1 if f[0] == "e" else 1 / 377)).astype(np.float32) for f in FIELDS}
    for wall in (False, True):  # a probe on a wall node takes source and probes out of the layer's launch
        pb.probes = np.array(cells + ([(0, 3), (2, 0)] if wall else []), np.int32)
        out = []
        for graph in (True, False):
            s = Sim.from_problem(pb, graph=graph)
            for f, a in init.items():
                s.set_field(f, a)
            s.step(7)
            s.step(33)
            got = {f: s.get_field(f) for f in FIELDS}
            got["probe"] = s.probe()
            out.append(got)
            s.close()
        o = O.for_problem(pb)
        o.set_state({f: a.astype(np.float64) for f, a in init.items()})
        rec = o.run(40)
        for f in FIELDS:
            assert rel_l2(out[0][f], getattr(o, f)) <= 1e-4, f
        assert rel_l2(out[0]["probe"], rec) <= 1e-4
        for k in out[0]:
            assert rel_l2(out[0][k], out[1][k]) <= 1e-5, k
