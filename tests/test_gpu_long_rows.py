"""Rows of more than 2^20 cells, which the 2D workgroup tiles do not take: the
marching kernels, the batch's marching passes and the adjoint's one-step
kernel (columns in pairs and single, with and without an absorbing layer,
loss and a mu_r map) against the oracle (relative L2 1e-4 for fields, loss
and gradients: runs this short are within 1e-6 of FP64)."""
import numpy as np
import pytest

from paper_2405_00814_amd import workloads as W

from helpers import log, rel_l2

pytestmark = pytest.mark.gpu
FIELDS = ("ez", "hx", "hy")
EVEN, ODD = (1 << 20) + 8, (1 << 20) + 9


def _problem(nx, ny, npml, T, maps=""):
    dt = 0.6e-3 / 2.99792458e8
    rng = np.random.default_rng(3)
    c = (nx // 2, ny // 2)
    box = (nx // 2 - 1, nx // 2 + 2, ny // 2 - 40, ny // 2 + 30)
    eps = np.ones((nx, ny), np.float32)
    eps[box[0]:box[1], box[2]:box[3]] = rng.uniform(1, 3, (3, 70))
    sig = mu = None
    if "s" in maps:
        sig = np.zeros((nx, ny), np.float32)
        sig[box[0]:box[1], box[2]:box[3]] = rng.uniform(0, 0.02, (3, 70))
    if "m" in maps:
        mu = np.ones((nx, ny), np.float32)
        mu[box[0]:box[1], box[2]:box[3]] = rng.uniform(1, 2, (3, 70))
    pb = W.Problem(name="long", ndim=2, shape=(nx, ny), dx=(1e-3, 1e-3), dt=dt, steps=T, npml=npml, eps_r=eps, sigma=sig,
                   mu_r=mu, source=W.Source(c, W.SRC_RICKER, (1.0, 6 * dt, 1.0 / (10 * dt))),
                   probes=np.array([(c[0] - 1, c[1] + 4), (c[0], c[1] - 5), (c[0], c[1] - 5), (c[0] + 1, c[1] + 33)], np.int32))
    return pb, box


@pytest.mark.parametrize("nx,ny,npml", [(8, EVEN, (0, 0, 8, 8)), (12, ODD, (3, 3, 8, 8)), (7, ODD, (0,) * 4)])
def test_stepping(nx, ny, npml):
    from oracle import oracle as O
    from paper_2405_00814_amd.sim import Batch, Sim
    pb, _ = _problem(nx, ny, npml, 26)
    o = O.for_problem(pb)
    rec = o.run(26)
    small = W.dielectric2d(70, ny=66, steps=26, seed=1, nrect=3, side=(6, 20), npml=8, nprobes=2)
    s, b = Sim.from_problem(pb), Batch([pb, small])
    assert s.get_kernel()["tile"][0] != 64
    for x in (s, b):
        x.step(3)
        x.step(23)
    for f in FIELDS:
        assert rel_l2(s.get_field(f), getattr(o, f)) <= 1e-4, f
        assert rel_l2(b.get_field(0, f), getattr(o, f)) <= 1e-4, f
    assert rel_l2(s.probe(), rec) <= 1e-4 and rel_l2(b.probe(0), rec) <= 1e-4
    s.close()
    b.close()


@pytest.mark.parametrize("nx,ny,npml,maps", [(8, EVEN, (0, 0, 8, 8), ""), (12, ODD, (3, 3, 8, 8), "sm"),
                                             (7, ODD, (0,) * 4, "s"), (8, EVEN, (0,) * 4, "m")])
def test_adjoint(nx, ny, npml, maps):
    from oracle import oracle as O
    from paper_2405_00814_amd.sim import Sim
    T = 24
    pb, box = _problem(nx, ny, npml, T, maps)
    ref = O.for_problem(pb).loss_and_grad(T, (8, T), box, mu="m" in maps)
    out = []
    for ckpt in (0, 7, T):
        s = Sim.from_problem(pb)
        r = s.adjoint_grads(T, (8, T), box, ckpt, mu="m" in maps)
        out.append([r[0]] + [g.cpu().numpy() for g in r[1:]])
        s.close()
    log("long rows", nx, ny, "loss", abs(out[0][0] / ref[0] - 1), "eps", rel_l2(out[0][1].reshape(ref[1].shape), ref[1]))
    for got in out:
        assert abs(got[0] - ref[0]) <= 1e-4 * abs(ref[0]) and ref[0] > 0
        assert rel_l2(got[1].reshape(ref[1].shape), ref[1]) <= 1e-4
        if "m" in maps:
            assert rel_l2(got[3].reshape(ref[2].shape), ref[2]) <= 1e-4
