"""Many probes in the 2D workgroup tiles: lines, blocks and repeated cells
give the record of the single-step kernel bit for bit, in every size class
and component, in the batch too; and a line of probes costs little."""
import numpy as np
import pytest

from paper_2405_00814_amd import workloads as W

pytestmark = pytest.mark.gpu


def _problem(shape, cells, npml=8):
    pb = W.dielectric2d(shape[0], ny=shape[1], steps=30, seed=1, nrect=6, side=(4, 24), npml=npml, nprobes=1)
    pb.source.cell = (shape[0] // 2, shape[1] // 2)
    pb.source.params = (1.0, 6 * pb.dt, 1.0 / (10 * pb.dt))
    pb.probes = np.array(cells, np.int32)
    return pb


def _cells(shape, kind):
    i, j = shape[0] // 2, shape[1] // 2
    if kind == "row":
        return [(i, q) for q in range(shape[1])]
    if kind == "column":
        return [(q, j + 1) for q in range(shape[0])][::-1]
    # a block with repeated cells, in no order
    c = [(i - 9 + a, j - 15 + b) for a in range(19) for b in range(31)] + [(i, j)] * 70
    return [c[q] for q in np.random.default_rng(4).permutation(len(c))]


@pytest.mark.parametrize("comp", ["ez", "hx", "hy"])
@pytest.mark.parametrize("kind", ["row", "column", "block"])
def test_records_of_the_single_step_kernel(kind, comp):
    from paper_2405_00814_amd.sim import Sim
    shape = (173, 140)
    pb = _problem(shape, _cells(shape, kind))
    pb.probe_component = comp
    out = []
    for kernel in ((2,), (3, (64, 0, 12)), (3, (64, 1, 7)), (3, (64, 2, 15))):
        s = Sim.from_problem(pb)
        s.set_kernel(*kernel)
        for n in (2, 17, 11):
            s.step(n)
        out.append(s.probe())
        s.close()
    assert np.abs(out[0]).max() > 0
    for r in out[1:]:
        assert np.array_equal(r, out[0])


def test_batch_records():
    from paper_2405_00814_amd.sim import Batch, Sim
    probs = [_problem(sh, _cells(sh, k)) for sh, k in (((173, 140), "block"), ((90, 201), "row"), ((66, 70), "column"))]
    b = Batch(probs)
    b.step(1)
    b.step(29)
    for q, pb in enumerate(probs):
        s = Sim.from_problem(pb)
        s.set_kernel(2)
        s.step(30)
        assert np.array_equal(b.probe(q), s.probe()), q
        s.close()
    b.close()


def test_cost_of_a_line_of_probes():
    """64 probes on a 64 x 64 cavity, the best of ten calls of 480 steps: a
    step with them takes less than twice one without (looked up one by one
    they made it 17 times as long; taken by the lanes of a wavefront they
    add two LDS reads)."""
    from paper_2405_00814_amd.sim import Sim
    t = []
    for cells in ([], [(32, q) for q in range(64)]):
        pb = W.cavity2d(64, steps=1, seed=0)
        pb.probes = np.array(cells, np.int32).reshape(-1, 2)
        s = Sim.from_problem(pb)
        best = 1e9
        for _ in range(10):
            s.step(480)
            best = min(best, s.last_step_time()[0])
        t.append(best)
        s.close()
    assert t[1] < 2.0 * t[0], t
