"""GPU parity of the adjoint's workgroup tiles: design boxes across tile and
wavefront seams and at the walls, absorbing layers, loss and mu_r maps, many
probes in one tile and several on one cell, both size classes: loss and
gradients against the oracle's discrete adjoint (bar 1e-4: the FP32 fields of
runs this short are within 1e-6 of FP64, and a gradient is a sum of products
of two of them), and the same bits for other checkpoint intervals."""
import numpy as np
import pytest

from paper_2405_00814_amd import workloads as W

from helpers import log, rel_l2

pytestmark = pytest.mark.gpu

CASES = [  # shape, npml, design, mat, mu, T
    ((70, 131), 8, (26, 50, 30, 100), 0, True, 130),
    ((90, 100), 0, (0, 24, 0, 44), 1, True, 120),
    ((90, 100), 0, (60, 90, 70, 100), 2, True, 120),
    ((33, 60), 0, (10, 20, 20, 40), 0, False, 90),
    ((430, 520), 12, (150, 260, 200, 330), 0, False, 90),
    ((430, 520), 12, (190, 260, 250, 300), 2, True, 90),
    ((520, 431), 12, (4, 80, 6, 70), 1, False, 90),
]


@pytest.mark.parametrize("shape,npml,design,mat,mu,T", CASES)
def test_adjoint_tiles_match_oracle(shape, npml, design, mat, mu, T):
    from oracle import oracle as O
    from paper_2405_00814_amd.sim import Sim
    i0, i1, j0, j1 = design
    rng = np.random.default_rng(4)
    pb = W.dielectric2d(shape[0], ny=shape[1], steps=T, seed=2, nrect=5, side=(4, 20), npml=npml, nprobes=1,
                        lossy=mat >= 1)
    pb.eps_r[i0:i1, j0:j1] = rng.uniform(1, 4, (i1 - i0, j1 - j0))
    if mat == 2:
        pb.mu_r = np.ones(shape, np.float32)
        pb.mu_r[i0:i1, j0:j1] = rng.uniform(1, 2, (i1 - i0, j1 - j0))
    c = ((i0 + i1) // 2, (j0 + j1) // 2)
    pb.source.cell = (max(1, c[0] - 3), max(1, c[1] - 2))
    pb.source.kind, pb.source.params = W.SRC_RICKER, (1.0, 30 * pb.dt, 1.0 / (25 * pb.dt))
    near = [(c[0] + a, c[1] + b) for a, b in ((0, 6), (1, 6), (1, 7), (5, -4), (5, -4), (-4, 0), (12, 9))]
    pb.probes = np.array([(min(shape[0] - 1, max(0, p)), min(shape[1] - 1, max(0, q))) for p, q in near], np.int32)
    window = (T // 3, T - 7)
    ref = O.for_problem(pb).loss_and_grad(T, window, design, mu=mu)
    out = []
    for ckpt in (0, 13, T):
        s = Sim.from_problem(pb)
        got = s.adjoint_grads(T, window, design, ckpt, mu=mu)
        out.append([got[0]] + [g.cpu().numpy() for g in got[1:]])
        s.close()
    loss, ge = out[0][0], out[0][1].reshape(ref[1].shape)
    log("adjoint tiles", shape, design, "loss", abs(loss / ref[0] - 1), "eps", rel_l2(ge, ref[1]))
    assert abs(loss - ref[0]) <= 1e-4 * abs(ref[0])
    assert rel_l2(ge, ref[1]) <= 1e-4
    if mu:
        assert rel_l2(out[0][3].reshape(ref[2].shape), ref[2]) <= 1e-4
    for o in out[1:]:
        assert o[0] == loss
        for a, b in zip(o[1:], out[0][1:]):
            assert np.array_equal(a, b)
