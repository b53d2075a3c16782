"""Calls on a live handle whose allocations fail (a caller's allocator that
returns NULL from the k-th call on): they return FDTD_ENOMEM, and the handle
steps on as if the call had not been made."""
import ctypes as C

import numpy as np
import pytest

from paper_2405_00814_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture
def budget(monkeypatch):
    """Allocations left to the library; None: no limit."""
    import torch
    from paper_2405_00814_amd import _lib as L
    from paper_2405_00814_amd import sim
    left = {"n": None}

    def alloc(ctx, size, stream):
        if left["n"] is not None:
            if left["n"] <= 0:
                return None
            left["n"] -= 1
        return int(torch.cuda.caching_allocator_alloc(int(size), stream=int(stream or 0)))

    def free(ctx, ptr, stream):
        torch.cuda.caching_allocator_delete(int(ptr))

    cb = L.ALLOC_FN(alloc), L.FREE_FN(free)
    a = L.fdtd_allocator(None, *cb)
    monkeypatch.setattr(sim, "torch_allocator", lambda: a)
    yield left
    left["n"] = None


def _fails_until_it_fits(left, call):
    """call() with room for 0, 1, ... allocations: FDTD_ENOMEM until it fits;
    yields after each failure with the limit lifted."""
    from paper_2405_00814_amd import _lib as L
    for k in range(60):
        left["n"] = k
        try:
            call()
        except L.FdtdError as e:
            assert e.code == L.FDTD_ENOMEM, e
            left["n"] = None
            yield k
            continue
        left["n"] = None
        return
    raise AssertionError("never fitted")


def _problem(ndim):
    if ndim == 2:
        return W.dielectric2d(96, ny=80, steps=40, seed=2, nrect=3, side=(6, 20), npml=8, nprobes=2)
    return W.yee3d(shape=(20, 22, 24), steps=40, seed=2, nbox=3, side=(3, 8), npml=4, nprobes=2, tau_steps=6.0)


def _state(s, fields):
    return [s.get_field(f) for f in fields] + [s.probe()]


@pytest.mark.parametrize("ndim", [2, 3])
def test_set_material_adding_loss(budget, ndim):
    """A box that makes a lossless grid lossy needs a Ca map."""
    from paper_2405_00814_amd.sim import Sim
    pb = _problem(ndim)
    pb.sigma = None
    fields = ("ez", "hx", "hy") if ndim == 2 else ("ex", "ey", "ez", "hx", "hy", "hz")
    lo, hi = (10,) * ndim, (16,) * ndim
    eps, sig = np.full((6,) * ndim, 2, np.float32), np.full((6,) * ndim, 0.02, np.float32)
    a, b = Sim.from_problem(pb), Sim.from_problem(pb)
    failed = 0
    a.step(20)
    b.step(20)
    for k in _fails_until_it_fits(budget, lambda: a.set_material(lo, hi, eps, sig)):
        failed += 1
        a.step(5)
        b.step(5)
        for u, v in zip(_state(a, fields), _state(b, fields)):
            assert np.array_equal(u, v), k
    assert failed
    b.set_material(lo, hi, eps, sig)
    for s in (a, b):
        s.step(15)
    for u, v in zip(_state(a, fields), _state(b, fields)):
        assert np.array_equal(u, v)
    a.close()
    b.close()


@pytest.mark.parametrize("split", [0, 1])
@pytest.mark.parametrize("shape", [(96, 80), (40, 36)])  # layers as runs of rows, and by CSR
def test_graph_set_material(budget, shape, split):
    """The layers are built again for new material: a rebuild that failed
    half-way is not stepped on."""
    from paper_2405_00814_amd.sim import Sim
    pb = W.dielectric2d(shape[0], ny=shape[1], steps=40, seed=2, nrect=3, side=(4, 12), npml=8, nprobes=2)
    pb.sigma = None
    pb.cpml = dict(m=3.0, sigma_max=0.0, kappa_max=1.0, alpha_max=0.0, m_alpha=1.0, split=split)
    a, b = (Sim.from_problem(pb, graph=True) for _ in range(2))
    lo, hi = (12, 12), (20, 20)
    eps, sig = np.full((8, 8), 2, np.float32), np.full((8, 8), 0.02, np.float32)
    failed = 0
    for s in (a, b):
        s.step(20)
    for k in _fails_until_it_fits(budget, lambda: a.set_material(lo, hi, eps, sig)):
        failed += 1
        for s in (a, b):
            s.step(3)
        for u, v in zip(_state(a, ("ez", "hx", "hy")), _state(b, ("ez", "hx", "hy"))):
            assert np.array_equal(u, v), k
    assert failed > 3
    b.set_material(lo, hi, eps, sig)
    for s in (a, b):
        s.step(15)
    for u, v in zip(_state(a, ("ez", "hx", "hy")), _state(b, ("ez", "hx", "hy"))):
        assert np.array_equal(u, v)
    a.close()
    b.close()


@pytest.mark.parametrize("form", ["reference", "tiles", "graph", "3d"])
def test_set_probes(budget, form):
    """New probes whose lists do not fit: the fields step on, and the call
    made again records from there."""
    from paper_2405_00814_amd.sim import Sim
    pb = _problem(3 if form == "3d" else 2)
    fields = ("ez", "hx", "hy")
    a, b = (Sim.from_problem(pb, graph=form == "graph") for _ in range(2))
    if form == "reference":
        for s in (a, b):
            s.set_kernel(1)
    cells = pb.probes + 1
    failed = 0
    for s in (a, b):
        s.step(20)
    for k in _fails_until_it_fits(budget, lambda: a.set_probes("ez", cells)):
        failed += 1
        for s in (a, b):
            s.step(3)
        for f in fields:
            assert np.array_equal(a.get_field(f), b.get_field(f)), (k, f)
    assert failed
    b.set_probes("ez", cells)
    for s in (a, b):
        s.step(9)
    for u, v in zip(_state(a, fields), _state(b, fields)):
        assert np.array_equal(u, v)
    a.close()
    b.close()


@pytest.mark.parametrize("cfg", [(4, 16, 1, 0), (2, 8, 2, 0), (1, 16, 1, 0)])
def test_batch_set_kernel_and_probes(budget, cfg):
    """A batch whose tile or probe lists did not fit builds them before it
    steps: no step is left out, no record written past its end."""
    from paper_2405_00814_amd.sim import Batch
    probs = W.batch2d(count=3, steps=0, seed=5, side=(70, 120), nprobes=5, rect_side=(8, 40), rect_density=40.0 / 4096)
    a, b = Batch(probs), Batch(probs)
    for x in (a, b):
        x.step(10)
    cells = probs[1].probes[:2]
    calls = [(lambda x: x.set_kernel(*cfg), 1e-5), (lambda x: x.set_probes(1, cells), 1e-5)]
    for call, tol in calls:
        failed = 0
        for k in _fails_until_it_fits(budget, lambda: call(a)):
            failed += 1
            a.step(13)
            b.step(13)
            for q in range(3):
                for f in ("ez", "hx", "hy"):
                    u, v = a.get_field(q, f), b.get_field(q, f)
                    assert np.linalg.norm(u - v) <= tol * np.linalg.norm(v), (k, q, f)
        assert failed
        call(b)
    for x in (a, b):
        x.step(9)
    for q in range(3):
        u, v = a.probe(q), b.probe(q)
        assert u.shape[0] == v.shape[0] == (2 if q == 1 else 5)
        assert np.allclose(u[:, -9:], v[:, -9:], rtol=1e-4, atol=1e-6 * np.abs(v).max()), q
    a.close()
    b.close()


@pytest.mark.parametrize("form", ["tiles", "single", "graph"])
def test_set_dft(budget, form):
    """A monitor whose arrays did not fit is no monitor."""
    from paper_2405_00814_amd import _lib as L
    from paper_2405_00814_amd.sim import Sim
    pb = _problem(2)
    a, b = (Sim.from_problem(pb, graph=form == "graph") for _ in range(2))
    if form == "single":
        for s in (a, b):
            s.set_kernel(2)
    for s in (a, b):
        s.step(20)
    mon = ("ez", (10, 12), (60, 50), [1e9, 2e9])
    failed = 0
    for k in _fails_until_it_fits(budget, lambda: a.set_dft(*mon)):
        failed += 1
        for s in (a, b):
            s.step(5)
        for u, v in zip(_state(a, ("ez", "hx", "hy")), _state(b, ("ez", "hx", "hy"))):
            assert np.array_equal(u, v), k
        with pytest.raises(L.FdtdError):
            a.get_dft()
    assert failed
    b.set_dft(*mon)
    for s in (a, b):
        s.step(31)
    assert np.array_equal(a.get_dft()[0], b.get_dft()[0])
    a.close()
    b.close()
