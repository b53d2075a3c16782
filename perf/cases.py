"""The work that programs built on this package have it do, as measurable
cases: time stepping of 2D and 3D grids (whole simulations from the zero
state), frequency-domain monitoring, the explicit graph form, batches of
uneven problems and gradients of a probe-energy loss.

``listed()`` names fixed cases, ``draw(rng)`` gives more of the same ranges.
``prepare`` makes what a program holds before the call (scene, handle,
output tensors), ``run`` is one pass through the public entry points,
``exact`` the same quantities in FP64 written out with plain torch.

The sources are zero-mean (a Ricker pulse, or a sine that keeps the fields
alive over the whole run); scenes, spatial steps and time steps follow the
package's workloads: random boxes, 20 cells per shortest wavelength at three
times the peak frequency, Courant number 0.99 of the limit.
"""
import math

import numpy as np
import torch

C0 = 299792458.0
MU0 = 1.25663706212e-6
EPS0 = 8.8541878128e-12
RICKER, SINE = 1, 3


def listed():
    return [
        # the smallest call: a tiny closed cavity, a few dozen steps (an
        # interactive program, a unit of a parameter sweep)
        dict(name="cavity_32", kind="grid2d", nx=32, ny=32, npml=0, scene="vacuum", f=15e9, src="sine",
             steps=64, nprobes=4, nf=0, form="grid"),
        # the resonance study of a small closed cavity, run to 1000 steps
        dict(name="cavity_128", kind="grid2d", nx=128, ny=128, npml=0, scene="vacuum", f=6e9, src="sine",
             steps=1000, nprobes=4, nf=0, form="grid"),
        # the smallest grid of the free-space timing sweep, absorbing layer
        # on every side
        dict(name="free_250", kind="grid2d", nx=250, ny=250, npml=16, scene="vacuum", f=1e9, src="sine",
             steps=1024, nprobes=1, nf=0, form="grid"),
        # a layered lossy body with a frequency-domain monitor over its lower
        # part and absorption rates from it
        dict(name="layered_400_monitor", kind="grid2d", nx=400, ny=400, npml=12, scene="layered", f=6.8e9,
             src="sine", steps=800, nprobes=4, nf=3, form="grid"),
        # a mid-size scene with odd sides and magnetic material
        dict(name="magnetic_1023x777", kind="grid2d", nx=1023, ny=777, npml=16, scene="magnetic", f=1e9,
             src="sine", steps=500, nprobes=6, nf=0, form="grid"),
        # the large 2D scene: lossy random rectangles, a line source, a
        # stretch of a long run
        dict(name="dielectric_4096", kind="grid2d", nx=4096, ny=4096, npml=16, scene="lossy", f=1e9,
             src="ricker", line=True, steps=400, nprobes=8, nf=0, form="grid"),
        # the explicit node-and-edge form of a 2D scene
        dict(name="graph_768", kind="grid2d", nx=768, ny=768, npml=16, scene="dielectric", f=1e9, src="sine",
             steps=200, nprobes=4, nf=0, form="graph"),
        # a small 3D volume with absorbing layers, ragged sides
        dict(name="yee_100x90x84", kind="grid3d", nx=100, ny=90, nz=84, npml=10, f=15e9, src="sine", steps=200,
             nprobes=4),
        # the large 3D volume, lit by a line source
        dict(name="yee_384", kind="grid3d", nx=384, ny=384, nz=384, npml=12, f=6e9, src="ricker", line=True,
             steps=40, nprobes=8),
        # many uneven 2D problems together, from their descriptions to their
        # probe records (a batch lives for one set of problems)
        dict(name="batch_16", kind="batch", count=16, lo=256, hi=900, npml=16, f=1e9, steps=3000, nprobes=4),
        # one gradient of an inverse-design loop, through autograd
        dict(name="adjoint_1024", kind="adjoint", nx=1024, ny=1024, npml=16, design=256, steps=1000, f=1e9,
             nprobes=16, mu=False, ckpt=0),
        # gradients with respect to eps_r, sigma and mu_r on a small odd grid,
        # every design value kept
        dict(name="adjoint_mu_211x260", kind="adjoint", nx=211, ny=260, npml=12, design=48, steps=600, f=1e9,
             nprobes=4, mu=True, ckpt=600),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    f = math.exp(rng.uniform(math.log(0.7e9), math.log(9e9)))
    pick = rng.random()
    if pick < 0.1:  # closed cavities
        n = _log(rng, 24, 180)
        return dict(kind="grid2d", nx=n, ny=_log(rng, 24, 180), npml=0, scene=rng.choice(["vacuum", "lossy"]), f=f,
                    src="sine", steps=_log(rng, 40, 1500), nprobes=rng.randint(1, 6), nf=0, form="grid")
    if pick < 0.45:  # 2D scenes of any size
        area = math.exp(rng.uniform(math.log(1.2e4), math.log(1.6e7)))
        r = math.exp(rng.uniform(-0.6, 0.6))
        nx, ny = max(70, int(math.sqrt(area * r))), max(70, int(math.sqrt(area / r)))
        steps = int(min(900, max(60, 4e9 / (nx * ny))) * rng.uniform(0.5, 1.0))
        nf = rng.choice([0, 0, 0, 1, 3]) if nx * ny < 2e6 else 0
        return dict(kind="grid2d", nx=nx, ny=ny, npml=rng.choice([8, 12, 16]),
                    scene=rng.choice(["vacuum", "dielectric", "lossy", "magnetic", "layered"]), f=f, src="sine",
                    line=rng.random() < 0.3, steps=steps, nprobes=rng.randint(1, 8), nf=nf, form="grid")
    if pick < 0.52:
        return dict(kind="grid2d", nx=_log(rng, 100, 900), ny=_log(rng, 100, 900), npml=rng.choice([8, 16]),
                    scene=rng.choice(["dielectric", "lossy"]), f=f, src="sine", steps=rng.randint(40, 200),
                    nprobes=rng.randint(1, 4), nf=0, form="graph")
    if pick < 0.72:  # 3D volumes
        vol = math.exp(rng.uniform(math.log(6e4), math.log(3e7)))
        e = vol ** (1.0 / 3.0)
        nx, ny, nz = (max(30, int(e * math.exp(rng.uniform(-0.3, 0.3)))) for _ in range(3))
        if rng.random() < 0.6:
            nz = max(32, nz // 4 * 4)
        return dict(kind="grid3d", nx=nx, ny=ny, nz=nz, npml=rng.choice([6, 10, 12]), f=6 * f, src="sine",
                    line=rng.random() < 0.5, steps=int(min(200, max(20, 1.2e9 / (nx * ny * nz)))), nprobes=rng.randint(1, 6))
    if pick < 0.86:
        lo = rng.randint(96, 300)
        return dict(kind="batch", count=rng.randint(4, 16), lo=lo, hi=lo + rng.randint(60, 500), npml=16, f=f,
                    steps=rng.randint(500, 2500), nprobes=rng.randint(1, 4))
    nx, ny = _log(rng, 120, 900), _log(rng, 120, 900)
    steps = rng.randint(200, 700)
    mu = rng.random() < 0.4
    return dict(kind="adjoint", nx=nx, ny=ny, npml=rng.choice([8, 12]), design=_log(rng, 16, min(nx, ny) // 4),
                steps=steps, f=f, nprobes=rng.randint(2, 12), mu=mu, ckpt=rng.choice([0, 0, 40, steps]))


# ---------------------------------------------------------------------------
# Scenes (host arrays, from the seed)
# ---------------------------------------------------------------------------

def _boxes(rng, shape, npml, count, lo, hi, a, vmax):
    """Axis-aligned boxes of random values in [1, vmax], clear of the layer."""
    for _ in range(count):
        sl = []
        for n in shape:
            inner = n - 2 * npml
            w = min(int(rng.integers(lo, hi + 1)), inner)
            p = int(rng.integers(npml, npml + inner - w + 1))
            sl.append(slice(p, p + w))
        a[tuple(sl)] = rng.uniform(1.0, vmax)


def _cell(rng, shape, margin, near=None, reach=0):
    """A cell clear of the layer; with near, within reach of that cell."""
    out = []
    for a, n in enumerate(shape):
        lo = min(margin, n // 3)
        hi = n - lo
        if near is not None:
            lo, hi = max(lo, min(hi - 1, near[a] - reach)), min(hi, max(lo + 1, near[a] + reach + 1))
        out.append(int(rng.integers(lo, max(hi, lo + 1))))
    return tuple(out)


def _line(c, shape, src):
    """First cell and (for a line along the first axis over half of the
    grid) last cell plus one of the source."""
    if not c.get("line"):
        return src, None
    n = shape[0]
    return (n // 4,) + src[1:], (3 * n // 4,) + tuple(v + 1 for v in src[1:])


def _scene2d(c, seed, nx=None, ny=None):
    """A dict of the plain inputs of a 2D problem."""
    rng = np.random.default_rng(seed)
    nx, ny = nx or c["nx"], ny or c["ny"]
    shape, npml, scene = (nx, ny), c["npml"], c.get("scene", "dielectric")
    emax = {"vacuum": 1.0, "layered": 45.0}.get(scene, 6.0)
    if scene == "vacuum" and npml == 0:
        h = 1e-3
    else:
        h = C0 / (3.0 * c["f"] * math.sqrt(emax) * 20)
    dt = 0.99 / math.sqrt(2.0) * h / C0
    eps = sig = mu = rho = None
    cells = nx * ny
    if scene in ("dielectric", "lossy", "magnetic"):
        eps = np.ones(shape, np.float32)
        nb = max(3, int(200 * cells / 4096 ** 2))
        _boxes(rng, shape, npml, nb, 8, max(12, min(shape) // 8), eps, 6.0)
        if scene == "lossy":
            sig = ((eps - 1.0) * np.float32(0.002)).astype(np.float32)
        if scene == "magnetic":
            mu = np.ones(shape, np.float32)
            _boxes(rng, shape, npml, nb, 8, max(12, min(shape) // 8), mu, 3.0)
    if scene == "layered":
        eps, sig, rho = np.ones(shape, np.float32), np.zeros(shape, np.float32), np.full(shape, 1.2, np.float32)
        edges = [int(v * nx) for v in (0.3, 0.34, 0.64)] + [nx]
        for k, (er, sg) in enumerate((((25, 45), (0.2, 0.5)), ((3, 8), (0.01, 0.05)), ((35, 45), (0.2, 0.4)))):
            eps[edges[k]:edges[k + 1]] = rng.uniform(*er)
            sig[edges[k]:edges[k + 1]] = rng.uniform(*sg)
            rho[edges[k]:edges[k + 1]] = rng.uniform(900, 1150)
    margin = npml + 8
    src = _cell(rng, shape, margin)
    if scene == "layered":
        src = (max(npml + 1, int(0.22 * nx)), ny // 2)
    src, hi = _line(c, shape, src)
    near = src if hi is None else ((src[0] + hi[0]) // 2,) + src[1:]
    probes = np.array([_cell(rng, shape, margin, near, max(4, c["steps"] // 4)) for _ in range(c["nprobes"])], np.int32)
    freqs = [c["f"] * (0.8 + 0.2 * q) for q in range(c.get("nf", 0))]
    box = ((int(0.31 * nx), npml), (nx - npml, ny - npml))
    return dict(shape=shape, dx=(h, h), dt=dt, eps=eps, sig=sig, mu=mu, rho=rho, npml=npml, src=src, hi=hi,
                probes=probes, kind=c.get("src", "ricker"), f=c["f"] if scene != "vacuum" else min(c["f"], C0 / (20 * h)),
                freqs=freqs, box=box)


def _scene3d(c, seed):
    rng = np.random.default_rng(seed)
    shape = (c["nx"], c["ny"], c["nz"])
    h = 1e-3
    dt = 0.99 / math.sqrt(3.0) * h / C0
    eps = np.ones(shape, np.float32)
    _boxes(rng, shape, c["npml"], max(60, int(500 * np.prod(shape) / 512 ** 3)), 4, max(8, min(shape) // 4), eps, 8.0)
    src = _cell(rng, shape, c["npml"] + 6)
    src, hi = _line(c, shape, src)
    near = src if hi is None else ((src[0] + hi[0]) // 2,) + src[1:]
    probes = np.array([_cell(rng, shape, c["npml"] + 4, near, max(3, c["steps"] // 8)) for _ in range(c["nprobes"])],
                      np.int32)
    # short runs: the pulse's peak falls inside the run
    f = 1.0 / (16 * dt) if c["src"] == "ricker" else min(c["f"], C0 / (10 * h))
    return dict(shape=shape, dx=(h, h, h), dt=dt, eps=eps, sig=None, mu=None, npml=c["npml"], src=src, hi=hi,
                probes=probes, kind=c["src"], f=f, freqs=[])


def _source(s):
    if s["kind"] == "ricker":
        return RICKER, (1.0, 1.5 / s["f"], s["f"])
    return SINE, (1.0, s["f"], 2.0 / s["f"])


def _problem(s, steps):
    from paper_2405_00814_amd import workloads as W
    nd = len(s["shape"])
    kind, par = _source(s)
    return W.Problem("case", nd, s["shape"], s["dx"], s["dt"], steps, (s["npml"],) * (2 * nd), s["eps"], s["sig"],
                     s["mu"], W.Source(s["src"], kind, par, hi=s["hi"]), s["probes"])


def _adjoint_scene(c, seed):
    rng = np.random.default_rng(seed)
    nx, ny, d = c["nx"], c["ny"], c["design"]
    h = C0 / (3.0 * c["f"] * 2.0 * 20)
    dt = 0.99 / math.sqrt(2.0) * h / C0
    i0, j0 = (nx - d) // 2, (ny - d) // 2
    box = (i0, i0 + d, j0, j0 + d)
    eps = np.ones((nx, ny), np.float32)
    eps[i0:i0 + d, j0:j0 + d] = rng.uniform(1.0, 4.0, (d, d))
    sig = mu = None
    if c["mu"]:
        sig, mu = np.zeros((nx, ny), np.float32), np.ones((nx, ny), np.float32)
        sig[i0:i0 + d, j0:j0 + d] = rng.uniform(0.0, 0.01, (d, d))
        mu[i0:i0 + d, j0:j0 + d] = rng.uniform(1.0, 2.0, (d, d))
    # source and probes in the ring between the absorbing layer and the box,
    # within a third of the grid's side of it
    near = max(4, min(nx, ny) // 6)

    def ring():
        while True:
            p = (int(rng.integers(max(c["npml"] + 2, i0 - near), min(nx - c["npml"] - 2, i0 + d + near))),
                 int(rng.integers(max(c["npml"] + 2, j0 - near), min(ny - c["npml"] - 2, j0 + d + near))))
            if not (i0 - 2 <= p[0] < i0 + d + 2 and j0 - 2 <= p[1] < j0 + d + 2):
                return p
    src = ring()
    probes = np.array([ring() for _ in range(c["nprobes"])], np.int32)
    return dict(shape=(nx, ny), dx=(h, h), dt=dt, eps=eps, sig=sig, mu=mu, npml=c["npml"], src=src, hi=None,
                probes=probes, kind="sine", f=c["f"], box=box, freqs=[])


def _batch_scenes(c, seed):
    rng, sizes = np.random.default_rng(seed), np.random.default_rng(c["count"] * 7919 + c["lo"])
    out = []
    for q in range(c["count"]):
        nx, ny = (int(sizes.integers(c["lo"], c["hi"] + 1)) for _ in range(2))
        out.append(_scene2d(dict(c, scene="dielectric", src="sine"), int(rng.integers(1 << 31)), nx, ny))
    return out


# ---------------------------------------------------------------------------
# One pass through the package
# ---------------------------------------------------------------------------

def prepare(case, seed):
    from paper_2405_00814_amd.sim import Sim
    c = case
    if c["kind"] == "batch":
        return dict(c=c, problems=[_problem(s, c["steps"]) for s in _batch_scenes(c, seed)])
    s = {"grid2d": _scene2d, "grid3d": _scene3d, "adjoint": _adjoint_scene}[c["kind"]](c, seed)
    graph = c.get("form") == "graph"
    sim = Sim.from_problem(_problem(s, c["steps"]), graph=graph)
    st = dict(c=c, sim=sim)
    if c["kind"] == "adjoint":
        i0, i1, j0, j1 = s["box"]
        st.update(box=s["box"], eps=torch.tensor(s["eps"][i0:i1, j0:j1], device="cuda"))
        return st
    if s["freqs"]:
        sim.set_dft("ez", s["box"][0], s["box"][1], s["freqs"])
        (a0, b0), (a1, b1) = s["box"]
        st["rho"] = None if s["rho"] is None else s["rho"][a0:a1, b0:b1]
    comps = ("ez", "hx", "hy") if len(s["shape"]) == 2 else ("ex", "ey", "ez", "hx", "hy", "hz")
    st["out"] = {k: None if graph else torch.empty(s["shape"], dtype=torch.float32, device="cuda") for k in comps}
    return st


def run(state):
    c = state["c"]
    if c["kind"] == "batch":
        from paper_2405_00814_amd.sim import Batch
        b = Batch(state["problems"])
        b.step(c["steps"])
        n = len(state["problems"])
        out = {"probe": [b.probe(q) for q in range(n)], "ez": [b.get_field(q, "ez") for q in range(n)]}
        b.close()
        return out
    sim = state["sim"]
    if c["kind"] == "adjoint":
        T = c["steps"]
        if c["mu"]:
            loss, ge, gs, gm = sim.adjoint_grads(T, (T // 2, T), state["box"], c["ckpt"], mu=True)
            return {"loss": np.float32(loss), "eps": ge, "sigma": gs, "mu": gm}
        from paper_2405_00814_amd.autograd import probe_energy_loss
        eps = state["eps"].clone().requires_grad_()
        loss = probe_energy_loss(sim, eps, T, (T // 2, T), state["box"], c["ckpt"])
        loss.backward()
        return {"loss": loss.detach().float(), "eps": eps.grad}
    sim.reset()
    sim.step(c["steps"])
    out = {"probe": sim.probe()}
    for k, t in state["out"].items():
        if t is None:
            out[k] = sim.get_field(k)
        else:
            sim.get_field_device(k, t)
            out[k] = t
    if c.get("nf"):
        x, _ = sim.get_dft()
        out["dft"] = x.astype(np.complex64)
        if state["rho"] is not None:
            out["sar"] = sim.dft_sar(state["rho"])
    return out


# ---------------------------------------------------------------------------
# Necessary work
# ---------------------------------------------------------------------------

def _maps(scene):
    return {"lossy": 2, "layered": 2, "magnetic": 2}.get(scene, 1)


def work(case):
    c = case
    if c["kind"] == "grid3d":
        n = c["nx"] * c["ny"] * c["nz"]
        # eps_r read once, six fields written once; 36 operations per cell
        # and step (six curls of four differences and two updates)
        return {"bytes": n * 4.0 * 7, "flops": 36.0 * n * c["steps"]}
    if c["kind"] == "batch":
        n = c["count"] * ((c["lo"] + c["hi"]) / 2.0) ** 2
        return {"bytes": n * 4.0 * 2, "flops": 13.0 * n * c["steps"]}
    n = c["nx"] * c["ny"]
    if c["kind"] == "adjoint":
        d = c["design"] ** 2
        # forward and transposed step, and two products per design cell
        return {"bytes": n * 4.0 + d * 4.0 * (3 if c["mu"] else 1),
                "flops": c["steps"] * (26.0 * n + (8.0 if c["mu"] else 4.0) * d)}
    b, fl = n * 4.0 * (_maps(c["scene"]) + 3), 13.0 * n * c["steps"]
    if c["nf"]:
        m = (c["nx"] - int(0.31 * c["nx"]) - c["npml"]) * (c["ny"] - 2 * c["npml"])
        b += m * c["nf"] * 8.0
        fl += m * c["nf"] * 4.0 * c["steps"]
    return {"bytes": b, "flops": fl}


# ---------------------------------------------------------------------------
# The same quantities in FP64 (plain torch)
# ---------------------------------------------------------------------------

def _axis(n, npml, d, dt, half, dev):
    """(1/d, b, c/d) of the absorbing layer's recursion along one axis,
    sigma graded with the third power of the depth, at i or i + 1/2."""
    x = torch.arange(n, dtype=torch.float64, device=dev) + (0.5 if half else 0.0)
    r = torch.zeros_like(x)
    if npml:
        r = torch.clamp((npml - x) / npml, min=0.0)
        r = torch.maximum(r, torch.clamp((x - (n - npml)) / npml, min=0.0))
    eta0 = math.sqrt(MU0 / EPS0)
    sg = 0.8 * 4.0 / (eta0 * d) * r ** 3
    b = torch.exp(-sg * dt / EPS0)
    cc = torch.where(sg > 0, b - 1.0, torch.zeros_like(b)) / d
    return 1.0 / d, b, cc


def _wave(s, n):
    t = (n + 1) * s["dt"]
    kind, par = _source(s)
    if kind == RICKER:
        a = (math.pi * par[2] * (t - par[1])) ** 2
        return par[0] * (1 - 2 * a) * math.exp(-a)
    w = math.sin(0.5 * math.pi * t / par[2]) ** 2 if t < par[2] else 1.0
    return par[0] * w * math.sin(2 * math.pi * par[1] * t)


def _src(s):
    """Index of the source's cells."""
    return s["src"] if s["hi"] is None else tuple(slice(a, b) for a, b in zip(s["src"], s["hi"]))


def _coef(s, eps, sig, mu):
    dt = s["dt"]
    sh = sig * dt / (2.0 * EPS0 * eps)
    return (1.0 - sh) / (1.0 + sh), dt / (EPS0 * eps) / (1.0 + sh), dt / (MU0 * mu)


def _map64(a, dev):
    return torch.tensor(1.0 if a is None else a, dtype=torch.float64, device=dev)


def _setup2d(s, dev):
    nx, ny = s["shape"]
    ax = {}
    for key, n, d, half in (("Ex", nx, s["dx"][0], 0), ("Hx", nx, s["dx"][0], 1), ("Ey", ny, s["dx"][1], 0),
                            ("Hy", ny, s["dx"][1], 1)):
        k, b, c = _axis(n, s["npml"], d, s["dt"], half, dev)
        ax[key] = (k, b[:, None], c[:, None]) if key[1] == "x" else (k, b[None, :], c[None, :])
    return ax


def _zeros2d(s, dev):
    nx, ny = s["shape"]
    z = lambda: torch.zeros(nx, ny, dtype=torch.float64, device=dev)  # noqa: E731
    return [z() for _ in range(7)]  # ez hx hy psi_hx psi_hy psi_ezx psi_ezy


def _pad_next(e, axis):
    z = torch.zeros_like(e.narrow(axis, 0, 1))
    return torch.cat((e.narrow(axis, 1, e.shape[axis] - 1), z), axis)


def _pad_prev(e, axis):
    z = torch.zeros_like(e.narrow(axis, 0, 1))
    return torch.cat((z, e.narrow(axis, 0, e.shape[axis] - 1)), axis)


def _step2d(st, ca, cb, db, ax, wall, src_mask, g):
    ez, hx, hy, phx, phy, pzx, pzy = st
    dy = _pad_next(ez, 1) - ez
    dx = _pad_next(ez, 0) - ez
    phx = ax["Hy"][1] * phx + ax["Hy"][2] * dy
    phy = ax["Hx"][1] * phy + ax["Hx"][2] * dx
    hx = hx - db * (ax["Hy"][0] * dy + phx)
    hy = hy + db * (ax["Hx"][0] * dx + phy)
    ddx = hy - _pad_prev(hy, 0)
    ddy = hx - _pad_prev(hx, 1)
    pzx = ax["Ex"][1] * pzx + ax["Ex"][2] * ddx
    pzy = ax["Ey"][1] * pzy + ax["Ey"][2] * ddy
    br = (ax["Ex"][0] * ddx + pzx) - (ax["Ey"][0] * ddy + pzy)
    ez = torch.where(wall, ez, ca * ez + cb * br) + g * src_mask
    return [ez, hx, hy, phx, phy, pzx, pzy]


def _fixed2d(s, dev):
    nx, ny = s["shape"]
    wall = torch.zeros(nx, ny, dtype=torch.bool, device=dev)
    wall[0], wall[:, 0] = True, True
    m = torch.zeros(nx, ny, dtype=torch.float64, device=dev)
    m[_src(s)] = 1.0
    pi = torch.tensor(s["probes"], device=dev, dtype=torch.long)
    return wall, m, pi


def _run2d(s, steps, dev):
    sig = torch.zeros((), dtype=torch.float64, device=dev) if s["sig"] is None else _map64(s["sig"], dev)
    ca, cb, db = _coef(s, _map64(s["eps"], dev), sig, _map64(s["mu"], dev))
    ax, st = _setup2d(s, dev), _zeros2d(s, dev)
    wall, m, pi = _fixed2d(s, dev)
    rec, acc = [], None
    if s["freqs"]:
        (a0, b0), (a1, b1) = s["box"]
        acc = torch.zeros(len(s["freqs"]), a1 - a0, b1 - b0, dtype=torch.complex128, device=dev)
    for n in range(steps):
        st = _step2d(st, ca, cb, db, ax, wall, m, _wave(s, n))
        rec.append(st[0][pi[:, 0], pi[:, 1]])
        if acc is not None:
            for q, f in enumerate(s["freqs"]):
                a = 2 * math.pi * f * (n + 1) * s["dt"]
                acc[q] += st[0][a0:a1, b0:b1] * complex(math.cos(a) * s["dt"], -math.sin(a) * s["dt"])
    return torch.stack(rec, 1), st, acc, sig


def _run3d(s, steps, dev):
    shape, dt = s["shape"], s["dt"]
    eps = _map64(s["eps"], dev)
    cb, db = dt / (EPS0 * eps), dt / MU0
    del eps
    ax = {}
    for a in range(3):
        for half in (0, 1):
            k, b, c = _axis(shape[a], s["npml"], s["dx"][a], dt, half, dev)
            v = [1, 1, 1]
            v[a] = -1
            ax[a, half] = (k, b.view(v), c.view(v))
    F = [torch.zeros(shape, dtype=torch.float64, device=dev) for _ in range(6)]  # ex ey ez hx hy hz
    lo, npml = {}, s["npml"]
    psi = {}

    def term(key, D, a, half):
        """The layer's difference along axis a: D/d, plus the recursion's
        value inside the two slabs."""
        k, b, c = ax[a, half]
        out = D * k
        if npml:
            n = shape[a]
            for side, st0, ln in ((0, 0, npml), (1, n - npml, npml)):
                d = D.narrow(a, st0, ln)
                bb, cc = b.narrow(a, st0, ln), c.narrow(a, st0, ln)
                p = psi.get((key, side))
                p = cc * d if p is None else bb * p + cc * d
                psi[key, side] = p
                out.narrow(a, st0, ln).add_(p)
        return out

    def dn(e, a):
        out = -e
        out.narrow(a, 0, shape[a] - 1).add_(e.narrow(a, 1, shape[a] - 1))
        return out

    def dp(h, a):
        out = h.clone()
        out.narrow(a, 1, shape[a] - 1).sub_(h.narrow(a, 0, shape[a] - 1))
        return out

    pi = torch.tensor(s["probes"], device=dev, dtype=torch.long)
    rec = []
    for n in range(steps):
        for h, (u, a, v, b) in enumerate(((1, 2, 2, 1), (2, 0, 0, 2), (0, 1, 1, 0))):
            F[3 + h].add_(term(("h", h, 0), dn(F[u], a), a, 1) - term(("h", h, 1), dn(F[v], b), b, 1), alpha=db)
        for e, (u, a, v, b) in enumerate(((5, 1, 4, 2), (3, 2, 5, 0), (4, 0, 3, 1))):
            br = cb * (term(("e", e, 0), dp(F[u], a), a, 0) - term(("e", e, 1), dp(F[v], b), b, 0))
            for axis in range(3):
                if axis != e:
                    br.narrow(axis, 0, 1).zero_()
            F[e].add_(br)
        F[2][_src(s)] += _wave(s, n)
        rec.append(F[2][pi[:, 0], pi[:, 1], pi[:, 2]])
    return torch.stack(rec, 1), F


def _adjoint(c, s, dev):
    from torch.utils.checkpoint import checkpoint
    T, (i0, i1, j0, j1) = c["steps"], s["box"]
    base = [_map64(s["eps"], dev), torch.zeros(s["shape"], dtype=torch.float64, device=dev) if s["sig"] is None
            else _map64(s["sig"], dev), torch.ones(s["shape"], dtype=torch.float64, device=dev) if s["mu"] is None
            else _map64(s["mu"], dev)]
    leaf = [m[i0:i1, j0:j1].clone().requires_grad_() for m in base]
    maps = []
    for m, p in zip(base, leaf):
        mask = torch.zeros(s["shape"], dtype=torch.bool, device=dev)
        mask[i0:i1, j0:j1] = True
        maps.append(m.masked_scatter(mask, p))
    ca, cb, db = _coef(s, *maps)
    ax, st = _setup2d(s, dev), _zeros2d(s, dev)
    wall, m, pi = _fixed2d(s, dev)

    def segment(k0, k1, ca, cb, db, *st):
        st, loss = list(st), torch.zeros((), dtype=torch.float64, device=dev)
        for n in range(k0, k1):
            st = _step2d(st, ca, cb, db, ax, wall, m, _wave(s, n))
            if n + 1 > T // 2:
                loss = loss + (st[0][pi[:, 0], pi[:, 1]] ** 2).sum()
        return (loss, *st)

    loss, L = 0.0, 32
    for k in range(0, T, L):
        part, *st = checkpoint(segment, k, min(T, k + L), ca, cb, db, *st, use_reentrant=False)
        loss = loss + part
    loss.backward()
    return loss.detach(), [p.grad for p in leaf]


def exact(case, seed):
    c, dev = case, "cuda" if torch.cuda.is_available() else "cpu"
    if c["kind"] == "batch":
        with torch.no_grad():
            ss = _batch_scenes(c, seed)
            # the whole batch would take too long: the first two problems
            got = [_run2d(s, c["steps"], dev)[:2] if q < 2 else None for q, s in enumerate(ss)]
        return {"probe": [None if g is None else g[0] for g in got], "ez": [None if g is None else g[1][0] for g in got]}
    if c["kind"] == "adjoint":
        s = _adjoint_scene(c, seed)
        loss, (ge, gs, gm) = _adjoint(c, s, dev)
        if c["mu"]:
            return {"loss": loss, "eps": ge.reshape(-1), "sigma": gs.reshape(-1), "mu": gm.reshape(-1)}
        return {"loss": loss, "eps": ge}
    with torch.no_grad():
        if c["kind"] == "grid3d":
            rec, F = _run3d(_scene3d(c, seed), c["steps"], dev)
            return dict(probe=rec, **dict(zip(("ex", "ey", "ez", "hx", "hy", "hz"), F)))
        s = _scene2d(c, seed)
        rec, st, acc, sig = _run2d(s, c["steps"], dev)
        out = dict(probe=rec, ez=st[0], hx=st[1], hy=st[2])
        if acc is not None:
            out["dft"] = acc
            if s["rho"] is not None:
                (a0, b0), (a1, b1) = s["box"]
                rho = _map64(s["rho"], dev)[a0:a1, b0:b1]
                out["sar"] = sig[a0:a1, b0:b1] * acc.abs() ** 2 / (2.0 * rho)
    return out
