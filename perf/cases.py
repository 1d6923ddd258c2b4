"""Workloads of the drop-particle library, for timing and for checking results.

Each case is one piece of work that a program asks of the library through its
Python entry points: a few lattice steps of a simulation (or an ensemble) with
its fields and particle records read back, or a pass of the surrogate network.
``listed`` gives the standing cases, ``draw`` others of the same ranges,
``prepare`` the objects a program holds before the call, ``run`` one pass,
``work`` the bytes and operations it cannot do without, and ``exact`` the same
outputs from a plain 64-bit evaluation of the method in torch.
"""
import math

import numpy as np
import torch

from paper_2505_10171_amd import workloads as W
from paper_2505_10171_amd.lbm import Context, Simulation
from paper_2505_10171_amd.surrogate import SRG_IN, SRG_OUT, Surrogate, flatten, he_init, unflatten

DEVICE = "cuda:0"


def listed():
    return [
        # the smallest box with everything in it (the first example, and the
        # unit of quick checks): launches and latency decide
        dict(name="sessile_drop_32", kind="drop", nx=32, ny=32, nz=32, spheres=1, radius=4.0,
             drop=10.0, touch=True, theta=90.0, force=0.0, ratio=1.0, storage="fp32", steps=40),
        # a sphere on a prescribed path through an interface (the capillary
        # detachment benchmark): each step a push, a step and the records
        dict(name="pulled_sphere_32x32x52", kind="pulled", nx=32, ny=32, nz=52, radius=10.0,
             theta=60.0, storage="fp32", steps=4),
        # a drop swept over spheres on the wall: the ordinary single run
        dict(name="drop_sweep_256x128x96", kind="drop", nx=256, ny=128, nz=96, spheres=20,
             radius=5.0, drop=30.0, touch=False, theta=110.0, force=5e-6, ratio=1.0,
             storage="fp32", steps=20),
        # the paper's own run (its Table 1): ragged sides, viscosity ratio 10
        dict(name="table1_400x181x71", kind="drop", nx=400, ny=181, nz=71, spheres=1, radius=10.0,
             drop=50.0, touch=False, theta=100.0, force=5e-6, ratio=10.0, storage="fp32",
             steps=20),
        # throughput at scale: the benchmark's slab with 500 spheres, the
        # largest box, in both population storages
        dict(name="slab_512x256x192", kind="slab", nx=512, ny=256, nz=192, spheres=500, radius=4.0,
             storage="fp32", steps=12),
        dict(name="slab_512x256x192_fp16", kind="slab", nx=512, ny=256, nz=192, spheres=500,
             radius=4.0, storage="fp16", steps=12),
        # pressure-driven flow between open ends in a tube with a sphere
        dict(name="tube_320x83x83", kind="tube", nx=320, tube=40.0, radius=12.2, storage="fp32",
             steps=20),
        # a drop on a wall with pillars, spheres between them
        dict(name="textured_256x128x64", kind="textured", nx=256, ny=128, nz=64, spheres=6,
             radius=4.0, drop=24.0, storage="fp32", steps=20),
        # many uneven boxes in one context, replayed from a graph (how the
        # surrogate's training runs are produced)
        dict(name="ensemble_64", kind="ensemble", members=64, storage="fp32", steps=40),
        # surrogate inference on a device batch, and for a handful of runs held
        # in host arrays
        dict(name="surrogate_predict_65536", kind="predict", rows=65536, host=False),
        dict(name="surrogate_predict_host_256", kind="predict", rows=256, host=True),
        # one epoch of surrogate training
        dict(name="surrogate_train_4096", kind="train", rows=4096, batch=256),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["drop", "drop", "slab", "slab", "tube", "textured", "pulled", "ensemble",
                       "predict", "train"])
    storage = rng.choice(["fp32", "fp32", "fp16"])
    if kind == "drop":
        nx, ny, nz = _log(rng, 28, 420), _log(rng, 28, 220), _log(rng, 28, 110)
        drop = rng.uniform(0.2, 0.35) * min(nx, ny, 2 * nz)
        small = min(nx, ny) < 64
        return dict(kind=kind, nx=nx, ny=ny, nz=nz, spheres=1 if small else rng.randint(1, 12),
                    radius=rng.uniform(3.0, 4.0 if small else 6.0), drop=drop, touch=small,
                    theta=rng.uniform(70.0, 115.0), force=rng.uniform(1e-6, 5e-6),
                    ratio=rng.choice([1.0, 10.0]), storage=storage, steps=rng.randint(8, 20))
    if kind == "slab":
        nx, ny, nz = _log(rng, 48, 512), _log(rng, 40, 256), _log(rng, 40, 192)
        return dict(kind=kind, nx=nx, ny=ny, nz=nz,
                    spheres=max(1, min(500, int(nx * ny * nz / 50000 * rng.uniform(0.3, 1.0)))),
                    radius=rng.uniform(3.0, 5.0), storage=storage, steps=rng.randint(6, 12))
    if kind == "tube":
        tube = rng.uniform(10.0, 40.0)
        return dict(kind=kind, nx=_log(rng, 64, 320), tube=tube,
                    radius=rng.uniform(0.25, 0.35) * tube, storage=storage,
                    steps=rng.randint(8, 20))
    if kind == "textured":
        return dict(kind=kind, nx=rng.randint(150, 256), ny=rng.randint(96, 128),
                    nz=rng.randint(48, 64), spheres=rng.randint(1, 6),
                    radius=rng.uniform(3.0, 4.0), drop=rng.uniform(16.0, 24.0), storage=storage,
                    steps=rng.randint(8, 20))
    if kind == "pulled":
        r = rng.uniform(5.0, 10.0)
        return dict(kind=kind, nx=rng.randint(26, 40), ny=rng.randint(26, 40),
                    nz=rng.randint(46, 60), radius=r, theta=rng.uniform(40.0, 130.0),
                    storage=storage, steps=rng.randint(2, 5))
    if kind == "ensemble":
        return dict(kind=kind, members=rng.randint(2, 64), storage=storage,
                    steps=2 * rng.randint(8, 20))
    if kind == "predict":
        return dict(kind=kind, rows=_log(rng, 1, 65536), host=rng.random() < 0.3)
    batch = 64 * rng.randint(1, 8)
    return dict(kind=kind, rows=batch * rng.randint(2, 8) + rng.randint(0, 63), batch=batch)


# ------------------------------------------------------------------ inputs
def _tanh_field(shape, dist, width=2.0):
    return torch.tanh(dist / width).to(torch.float32).expand(shape).contiguous().cpu().numpy()


def _axes(nx, ny, nz):
    ax = [torch.arange(n, dtype=torch.float64, device=DEVICE) for n in (nx, ny, nz)]
    return ax[0][None, None, :], ax[1][None, :, None], ax[2][:, None, None]


def _drop_phi0(nx, ny, nz, centre, radius):
    x, y, z = _axes(nx, ny, nz)
    dx, dy = x - centre[0], y - centre[1]
    dx, dy = dx - nx * torch.round(dx / nx), dy - ny * torch.round(dy / ny)
    r = torch.sqrt(dx * dx + dy * dy + (z - centre[2]) ** 2)
    return _tanh_field((nz, ny, nx), radius - r)


def _scatter(g, count, lo, hi, period, gap, allowed=lambda p: True, first=()):
    """Up to `count` seeded positions in [lo, hi] at least `gap` apart, `first` among them."""
    pts = np.array(first).reshape(-1, 3)
    for _ in range(400 * count):
        if len(pts) == count:
            break
        p = g.uniform(lo, hi)
        d = pts - p
        d -= period * np.round(d / period)
        if (not len(pts) or (d * d).sum(axis=1).min() >= gap * gap) and allowed(p):
            pts = np.vstack([pts, p])
    return pts


def _sims(case, seed):
    """The simulations (cfg, phi0, particles) of a lattice case."""
    g = W.rng(seed, 0)
    kind = case["kind"]
    if kind == "ensemble":
        sims = []
        for i in range(case["members"]):
            gi = W.rng(seed, i)
            side = int(W.rng(4, i).choice([48, 64, 80, 96]))  # the boxes are the case's, not the seed's
            R = gi.uniform(3.0, 6.0)
            Rc = R + W.DEFAULTS["delta_R"]
            Rd = gi.uniform(12.0, min(24.0, (side - 2 * Rc - 8) / 2.0))
            cfg = W.config(side, side, side, body_force=(gi.uniform(1e-6, 1e-5), 0.0, 0.0),
                           storage=case["storage"])
            p = W.particle((side / 4.0 + Rd + Rc + 2.0, side / 2.0 + gi.uniform(-0.5, 0.5),
                            0.5 + Rc), R, theta_deg=gi.uniform(30.0, 150.0),
                           mu_s=gi.uniform(0.0, 1.0), mu_r=gi.uniform(0.0, 0.1))
            phi0 = _drop_phi0(side, side, side, (side / 4.0, side / 2.0, 0.5), Rd)
            sims.append(dict(cfg=cfg, phi0=phi0, particles=[p]))
        return sims
    if kind == "tube":
        R_t, R, nx = case["tube"], case["radius"], case["nx"]
        ny = nz = int(2 * R_t) + 3
        rho, nu, v = 1.05, 0.457, 0.0113
        half = 0.5 * 3.0 * 8.0 * rho * nu * v * nx / (R_t * R_t)
        half = min(half, 0.05 * rho)
        cfg = W.config(nx, ny, nz, has_wall=2, tube_R=R_t, open_x=1, rho0=rho, rho_in=rho + half,
                       rho_out=rho - half, tau_a=0.5 + 3 * nu, tau_b=0.5 + 3 * nu, sigma=0.0,
                       storage=case["storage"])
        a, off = g.uniform(0.0, 2.0 * np.pi), 0.21 * R_t
        # released with the mean flow
        p = W.particle((max(0.25 * nx, R + 8.0), 0.5 * (ny - 1) + off * np.cos(a),
                        0.5 * (nz - 1) + off * np.sin(a)), R, rho_p=rho, g_p=0.0, mu_s=0.0,
                       mu_r=0.0, v=(v, 0.0, 0.0))
        return [dict(cfg=cfg, phi0=None, particles=[p])]
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    R = case["radius"]
    if kind == "pulled":
        cfg = W.config(nx, ny, nz, storage=case["storage"])
        z_int = 0.43 * nz
        x, y, z = _axes(nx, ny, nz)
        phi0 = _tanh_field((nz, ny, nx), z_int - z)
        p = W.particle((nx / 2.0 + g.uniform(-0.5, 0.5), ny / 2.0 + g.uniform(-0.5, 0.5),
                        z_int - R * math.cos(math.radians(case["theta"]))), R,
                       theta_deg=case["theta"], kinematic=1)
        return [dict(cfg=cfg, phi0=phi0, particles=[p])]
    Rc = R + W.DEFAULTS["delta_R"]
    if kind == "slab":
        cfg = W.config(nx, ny, nz, storage=case["storage"])
        x, y, z = _axes(nx, ny, nz)
        phi0 = _tanh_field((nz, ny, nx), 0.4 * nz - z)
        pts = _scatter(g, case["spheres"], [0.0, 0.0, 0.5 + Rc], [nx, ny, nz - 0.5 - Rc],
                       np.array([nx, ny, 1e9]), 2 * Rc + 1,
                       # one in the interface whatever their number
                       first=g.uniform([0.0, 0.0, 0.4 * nz - 1.0], [nx, ny, 0.4 * nz + 1.0]))
        parts = [W.particle((p[0] % nx, p[1] % ny, p[2]), R) for p in pts]
        return [dict(cfg=cfg, phi0=phi0, particles=parts)]
    if kind == "textured":
        sx, sy = nx / 5.33, ny / 2.67
        boxes = [(int(sx * (i + 1)) - 6, int(0.5 * ny + sy * (j - 0.5)) - 6, 1,
                  int(sx * (i + 1)) + 5, int(0.5 * ny + sy * (j - 0.5)) + 5, 8)
                 for i in range(4) for j in range(2)]
        cfg = W.config(nx, ny, nz, has_wall=3, boxes=boxes, theta_wall_deg=110.0,
                       body_force=(4e-6, 0.0, 0.0), storage=case["storage"])
        Rd = case["drop"]
        phi0 = _drop_phi0(nx, ny, nz, (1.5 * sx, 0.5 * ny, 8.5), Rd)

        def clear(p):
            return all(max(b[0] - 0.5 - p[0], p[0] - b[3] - 0.5, b[1] - 0.5 - p[1],
                           p[1] - b[4] - 0.5) > Rc + 1.0 for b in boxes)
        pts = _scatter(g, case["spheres"], [1.5 * sx + Rd + Rc + 10.0, Rc, 0.5 + Rc],
                       [nx - Rc, ny - Rc, 0.5 + Rc], np.array([nx, ny, 1e9]), 2 * Rc + 1, clear)
        parts = [W.particle(p, R, theta_deg=g.uniform(60.0, 120.0)) for p in pts]
        return [dict(cfg=cfg, phi0=phi0, particles=parts)]
    # a drop on the wall, pushed along x, spheres on the wall
    tau = {} if case["ratio"] == 1.0 else dict(tau_a=W.TAU_DROP, tau_b=W.TAU_AIR)
    cfg = W.config(nx, ny, nz, theta_wall_deg=case["theta"],
                   body_force=(case["force"], 0.0, 0.0), storage=case["storage"], **tau)
    Rd, c = case["drop"], np.array([0.25 * nx, 0.5 * ny])
    if case["touch"]:  # the sphere at the drop's contact line
        c[0] = 0.45 * nx
        pts = [np.array([c[0] + Rd + g.uniform(-0.5, 0.5), c[1], 0.5 + Rc])]
    else:
        def clear(p):
            d = p[:2] - c
            d -= np.array([nx, ny]) * np.round(d / np.array([nx, ny]))
            return math.hypot(*d) >= Rd + Rc + 10.0
        pts = _scatter(g, case["spheres"], [0.0, 0.0, 0.5 + Rc], [nx, ny, 0.5 + Rc],
                       np.array([nx, ny, 1e9]), 2 * Rc + 1, clear)
    parts = [W.particle((p[0] % nx, p[1] % ny, p[2]), R, theta_deg=g.uniform(30.0, 120.0),
                        mu_s=g.uniform(0.0, 1.0), mu_r=g.uniform(0.0, 0.1),
                        g_p=10.0 * cfg["sigma"] * R) for p in pts]
    return [dict(cfg=cfg, phi0=_drop_phi0(nx, ny, nz, (c[0], c[1], 0.5), Rd), particles=parts)]


def _path(p, k):
    """The prescribed path of a pulled sphere: up and down about its start."""
    w = 2.0 * math.pi / 400.0
    return dict(p, x=(p["x"][0], p["x"][1], p["x"][2] + 0.6 * math.sin(w * k)),
                v=(0.0, 0.0, 0.6 * w * math.cos(w * k)))


def _set(case, seed):
    """A training set: parameters, outcome labels and trajectories, standardised."""
    g = W.rng(seed, 1)
    X = g.standard_normal((case["rows"], SRG_IN)).astype(np.float32)
    traj = np.tanh(X @ g.standard_normal((SRG_IN, 48)) / 2.0) + 0.1 * g.standard_normal(
        (case["rows"], 48))
    label = np.argmax(X @ g.standard_normal((SRG_IN, 3)), axis=1).astype(np.int32)
    return X, label, traj.astype(np.float32)


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("predict", "train"):
        n = case["rows"]
        s = Surrogate(max_batch=max(64, -(-n // 64) * 64), max_train=n, device=DEVICE)
        s.set_params(flatten(he_init(seed)))
        if kind == "train":
            s.set_train(*_set(case, seed))
            return dict(case=case, net=s)
        X = W.rng(seed, 1).standard_normal((n, SRG_IN)).astype(np.float32)
        if case["host"]:
            return dict(case=case, net=s, X=X)
        return dict(case=case, net=s, X=torch.from_numpy(X).to(DEVICE),
                    y=torch.empty(n, SRG_OUT, device=DEVICE))
    sims = _sims(case, seed)
    if kind == "ensemble":
        stream = torch.cuda.Stream()
        ctx = Context(sims, device=DEVICE, stream=stream)
        ctx.use_graph(True)
        return dict(case=case, ctx=ctx, stream=stream)
    sim = Simulation(sims[0]["cfg"], sims[0]["phi0"], sims[0]["particles"], device=DEVICE)
    return dict(case=case, ctx=sim, parts=sims[0]["particles"], k=0)


# -------------------------------------------------------------------- runs
LOG = ("x", "v", "F_hyd", "F_cap")


def _log_records(parts):
    """A run's log of its particles, in single precision (what the FP32 and
    FP16 lattices resolve of the forces): one array per quantity."""
    return {k: np.array([p[k] for p in parts], np.float32) for k in LOG}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "predict":
        if case["host"]:
            return state["net"].predict(state["X"])
        state["net"].predict_device(state["X"], state["y"])
        return state["y"]
    if kind == "train":
        loss = state["net"].train(1, batch=case["batch"], lr=1e-3, seed=1)
        return dict(loss=loss, params=state["net"].get_params())
    ctx = state["ctx"]
    if kind == "pulled":
        log = []
        for _ in range(case["steps"]):
            ctx.push_particles([_path(p, state["k"]) for p in state["parts"]])
            ctx.step(1)
            state["k"] += 1
            log.append(ctx.particles()[0])
        rho, u, phi = ctx.fields_device()
        return dict(rho=rho, u=u, phi=phi, **_log_records(log))
    ctx.step(case["steps"])
    if kind == "ensemble":
        fields = [ctx.fields_device(i) for i in range(ctx.n)]
        log = _log_records([ctx.particles(i)[0] for i in range(ctx.n)])
        return dict(rho=torch.cat([f[0] for f in fields]), u=torch.cat([f[1] for f in fields]),
                    phi=torch.cat([f[2] for f in fields]), **log)
    rho, u, phi = ctx.fields_device()
    return dict(rho=rho, u=u, phi=phi, **_log_records(ctx.particles()))


def work(case):
    kind = case["kind"]
    net = sum(a * b for a, b in ((6, 256), (256, 256), (256, 256), (256, 256), (256, 51)))
    if kind == "predict":
        return dict(bytes=4.0 * case["rows"] * (SRG_IN + SRG_OUT) + 2.0 * net,
                    flops=2.0 * net * case["rows"])
    if kind == "train":
        n = case["rows"] // case["batch"]
        # forward and two backward products per sample; per batch the weights'
        # gradients, moments and values once
        return dict(bytes=n * (28.0 * net + 4.0 * case["batch"] * 55),
                    flops=6.0 * net * n * case["batch"])
    if kind == "tube":
        side = int(2 * case["tube"]) + 3
        nodes = math.pi * case["tube"] ** 2 / side ** 2 * case["nx"] * side * side
    elif kind == "ensemble":
        nodes = case["members"] * (48.0 ** 3 + 64.0 ** 3 + 80.0 ** 3 + 96.0 ** 3) / 4.0
    else:
        nodes = float(case["nx"] * case["ny"] * case["nz"])
    # per node-step the 19 total populations read and written once, the order
    # parameter read and written once, the mask read; the read-out at the end
    p = 2 if case["storage"] == "fp16" else 4
    return dict(bytes=nodes * (case["steps"] * (38.0 * p + 10.0) + 20.0 + 19.0 * p),
                flops=nodes * case["steps"] * 400.0)


# ------------------------------------------------------ 64-bit evaluation
C = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1),
     (1, 1, 0), (1, -1, 0), (-1, 1, 0), (-1, -1, 0), (1, 0, 1), (1, 0, -1), (-1, 0, 1),
     (-1, 0, -1), (0, 1, 1), (0, 1, -1), (0, -1, 1), (0, -1, -1)]
OPP = [C.index((-a, -b, -c)) for a, b, c in C]
WQ = [1 / 3 if c == (0, 0, 0) else 1 / 18 if sum(map(abs, c)) == 1 else 1 / 36 for c in C]
EPS = 1e-4  # threshold of the normal and of the wetting rotation's tangential part


def _shift(a, i):
    """a at x + c_i (z, y, x order)."""
    cx, cy, cz = C[i]
    return torch.roll(a, (-cz, -cy, -cx), (0, 1, 2))


def _dot(i, v):
    """c_i . v of three fields."""
    return sum(c * a for c, a in zip(C[i], v) if c) if i else 0.0


def _cross(a, b):
    return torch.linalg.cross(a, b, dim=-1)


class Exact:
    """One simulation of the coupled method in 64 bits (arXiv 2505.10171:
    colour-gradient lattice Boltzmann with moving bounce-back, wetting,
    capillary forces and DEM), as whole-array torch."""

    def __init__(self, sim):
        c = self.c = sim["cfg"]
        self.shape = (c["nz"], c["ny"], c["nx"])
        t = self.t = lambda a: torch.as_tensor(np.array(a, np.float64), device=DEVICE)
        self.L = t([c["nx"], c["ny"], c["nz"]])
        z, y, x = torch.meshgrid(*[torch.arange(n, device=DEVICE) for n in self.shape],
                                 indexing="ij")
        wall = torch.zeros(self.shape, dtype=torch.bool, device=DEVICE)
        if c["has_wall"] in (1, 3):
            wall |= z == 0
        if c["has_wall"] == 3:
            for b in c["boxes"]:
                wall[b[2]:b[5] + 1, b[1]:b[4] + 1, b[0]:b[3] + 1] = True
        if c["has_wall"] == 2:
            wall |= ((y - 0.5 * (c["ny"] - 1)) ** 2 + (z - 0.5 * (c["nz"] - 1)) ** 2
                     >= c["tube_R"] ** 2)
        self.wall, self.xs = wall, x
        ps = sim["particles"]
        self.n = len(ps)
        rec = {k: t([p[k] for p in ps]) for k in ("x", "v", "w", "R", "rho_p", "mu_s", "mu_r",
                                                  "g_p", "theta_deg")}
        self.__dict__.update({"p_" + k: v for k, v in rec.items()})
        self.kin = torch.tensor([bool(p["kinematic"]) for p in ps], device=DEVICE)
        self.mass = self.p_rho_p * 4.0 / 3.0 * math.pi * self.p_R ** 3
        self.inertia = 0.4 * self.mass * self.p_R ** 2
        self.Rc = self.p_R + c["delta_R"]
        m = sorted(self.mass.tolist())
        eff = m[0] * m[1] / (m[0] + m[1]) if self.n > 1 else m[0]
        tc = math.pi / math.sqrt(c["kn"] / eff - (c["gn"] / (2 * eff)) ** 2)
        self.n_sub = max(1, math.ceil(45.0 / tc))
        zero = torch.zeros(self.n, 3, dtype=torch.float64, device=DEVICE)
        self.Fh = self.Fc = self.Fcp = self.Tcp = zero
        self.prev = None
        self.walls = {1: 2, 2: 1, 3: 2 + len(c.get("boxes", ()))}.get(c["has_wall"], 0)
        self.xt = zero.new_zeros(self.n, self.n + self.walls, 3)
        self.xr = self.xt.clone()
        self.mask = self._mask()
        phi0 = (torch.ones(self.shape, dtype=torch.float64, device=DEVICE)
                if sim["phi0"] is None else t(sim["phi0"]))
        w = t(WQ)[:, None, None, None]
        self.f = (w * c["rho0"]).expand(19, *self.shape).clone()
        self.g = self.f * phi0
        self._links()

    # -------------------------------------------------------------- solids
    def _mask(self):
        m = torch.full(self.shape, 1 << 20, dtype=torch.int64, device=DEVICE).view(-1)
        B = int(math.ceil(2 * self.p_R.max().item())) + 4
        o = torch.arange(B, device=DEVICE)
        lo = torch.floor(self.p_x - self.p_R[:, None]).long() - 1
        idx, d2 = 0, 0.0
        n = [self.shape[2], self.shape[1], self.shape[0]]
        stride = (1, n[0], n[0] * n[1])
        for k in range(3):
            a = lo[:, k, None] + o
            view = [self.n, 1, 1, 1]
            view[1 + k] = B
            d = a.double() - self.p_x[:, k, None]
            idx = idx + ((a % n[k]) * stride[k]).view(view)
            d2 = d2 + (d * d).view(view)
        inside = d2 < (self.p_R ** 2).view(-1, 1, 1, 1)
        code = torch.arange(2, self.n + 2, device=DEVICE).view(-1, 1, 1, 1).expand(inside.shape)
        m.scatter_reduce_(0, idx.expand(inside.shape)[inside], code[inside], "amin")
        m[m == 1 << 20] = 0
        m = m.view(self.shape)
        return torch.where(self.wall, torch.ones_like(m), m)

    def _links(self):
        """Per direction: the neighbour is solid, or beyond an open end."""
        solid = self.mask != 0
        self.fluid = ~solid
        self.out = [None] * 19
        self.blocked = [None] * 19
        for i in range(1, 19):
            b = _shift(solid, i)
            if self.c.get("open_x") and C[i][0]:
                edge = 0 if C[i][0] < 0 else self.shape[2] - 1
                self.out[i] = self.xs == edge
                b = b | self.out[i]
            self.blocked[i] = b

    def _gradient(self, a):
        """3 sum_i w_i c_i a(x + c_i), the value at x for a blocked neighbour."""
        G = [torch.zeros_like(a) for _ in range(3)]
        for i in range(1, 19):
            v = torch.where(self.blocked[i], a, _shift(a, i))
            for k in range(3):
                if C[i][k]:
                    G[k] += (3.0 * WQ[i] * C[i][k]) * v
        return G

    def _wall_normal(self, x):
        """The static wall's normal at nodes x (m x 3)."""
        c, n = self.c, torch.zeros_like(x)
        if c["has_wall"] == 1:
            n[:, 2] = torch.where(x[:, 2] == 1, 1.0, -1.0)
        elif c["has_wall"] == 2:
            n[:, 1:] = 0.5 * (self.L[1:] - 1) - x[:, 1:]
            n = n / n.norm(dim=1, keepdim=True).clamp_min(1e-300)
        elif c["has_wall"] == 3:
            top, under = x[:, 2] - 0.5, c["nz"] - 0.5 - x[:, 2]
            best = torch.minimum(top, under)
            n[:, 2] = torch.where(top <= under, 1.0, -1.0)
            for b in c["boxes"]:
                d = x - torch.minimum(torch.maximum(x, self.t(b[:3]) - 0.5), self.t(b[3:]) + 0.5)
                r = d.norm(dim=1)
                near = (r > 0) & (r < best)
                best = torch.where(near, r, best)
                n = torch.where(near[:, None], d / r.clamp_min(1e-300)[:, None], n)
        return n

    def _interface(self):
        """phi, normal, |G|, CSF and body force of the current state."""
        c = self.c
        phi = torch.where(self.fluid, self.g.sum(0) / self.f.sum(0), 0.0)
        G = self._gradient(phi)
        far = 1 << 20
        part = torch.full(self.shape, far, device=DEVICE)
        wet = torch.zeros_like(self.wall)
        for i in range(1, 19):
            nb = _shift(self.mask, i)
            if self.out[i] is not None:
                nb = torch.where(self.out[i], 0, nb)
            wet |= nb == 1
            part = torch.minimum(part, torch.where(nb >= 2, nb - 2, far))
        g = torch.sqrt(G[0] ** 2 + G[1] ** 2 + G[2] ** 2)
        at = (self.fluid & (wet | (part < far)) & (g > EPS)).nonzero(as_tuple=True)
        if len(at[0]):
            x = torch.stack([at[2], at[1], at[0]], 1).double()
            p = part[at]
            hit = p < far
            p = torch.where(hit, p, 0)
            d = self._image(x - self.p_x[p])
            ns = torch.where(hit[:, None], d / d.norm(dim=1, keepdim=True), self._wall_normal(x))
            th = torch.where(hit, self.p_theta_deg[p],
                             torch.full_like(d[:, 0], c["theta_wall_deg"])) * math.pi / 180.0
            v = torch.stack([a[at] for a in G], 1)
            gm = g[at]
            tan = v - (v * ns).sum(1, keepdim=True) * ns
            tn = tan.norm(dim=1)
            rot = gm[:, None] * (-torch.cos(th)[:, None] * ns
                                 + torch.sin(th)[:, None] * tan / tn.clamp_min(1e-300)[:, None])
            wgt = ((tn / EPS - 1.0).clamp(0.0, 1.0) * (gm / EPS - 1.0).clamp(0.0, 1.0))[:, None]
            v = torch.where(tn[:, None] > EPS, v + wgt * (rot - v), v)
            for k in range(3):
                G[k][at] = v[:, k]
        g = torch.sqrt(G[0] ** 2 + G[1] ** 2 + G[2] ** 2)
        big = g.clamp_min(EPS)
        n = [torch.where(self.fluid, a / big, 0.0) for a in G]
        del G
        kappa = sum(self._gradient(n[k])[k] for k in range(3))
        F = [-0.5 * c["sigma"] * kappa * big * n[k] + c["body_force"][k] * 0.5 * (1.0 + phi)
             for k in range(3)]
        return phi, n, big, F

    def _velocity(self, F):
        rho = self.f.sum(0)
        j = [torch.zeros_like(rho) for _ in range(3)]
        for i in range(1, 19):
            for k in range(3):
                if C[i][k]:
                    j[k] += C[i][k] * self.f[i]
        return rho, [(j[k] + 0.5 * F[k]) / rho for k in range(3)]

    def _image(self, d):
        return d - self.L * torch.ceil(d / self.L - 0.5)

    # ---------------------------------------------------------------- step
    def step(self):
        c = self.c
        phi, n, big, F = self._interface()
        rho, u = self._velocity(F)
        self._capillary(phi, n, big)
        uu = u[0] ** 2 + u[1] ** 2 + u[2] ** 2
        uF = u[0] * F[0] + u[1] * F[1] + u[2] * F[2]
        nua, nub = (c["tau_a"] - 0.5) / 3.0, (c["tau_b"] - 0.5) / 3.0
        om = 1.0 / (0.5 + 3.0 / ((1 + phi) / (2 * nua) + (1 - phi) / (2 * nub)))
        om2 = 8.0 * (2.0 - om) / (8.0 - om)
        ks, ka = 1.0 - 0.5 * om, 1.0 - 0.5 * om2
        f = self.f
        for i in [0] + [i for i in range(1, 19) if i < OPP[i]]:
            o = OPP[i]
            cu, cF = _dot(i, u), _dot(i, F)
            sy = 0.5 * (f[i] + f[o]) - WQ[i] * rho * (1.0 + 4.5 * cu * cu - 1.5 * uu)
            even = -om * sy + ks * WQ[i] * (9.0 * cu * cF - 3.0 * uF)
            if i == 0:
                f[0] += even
                continue
            an = 0.5 * (f[i] - f[o]) - 3.0 * WQ[i] * rho * cu
            odd = -om2 * an + ka * 3.0 * WQ[i] * cF
            f[i] += even + odd
            f[o] += even - odd
        r = 0.5 * c["beta"] * rho * (1.0 - phi * phi)
        self.g[0] = phi * f[0]
        new = torch.empty_like(f)
        new[0] = f[0]
        Fh = torch.zeros(self.n, 3, dtype=torch.float64, device=DEVICE)
        Th = Fh.clone()
        for i in range(1, 19):
            o, b = OPP[i], self.blocked[OPP[i]]
            seg = WQ[i] * r * _dot(i, n)
            new[i] = torch.where(b, f[o], _shift(f[i], o))
            self.g[i] = torch.where(b, phi * f[o] - seg, _shift(phi * f[i] + seg, o))
            if self.out[o] is not None:
                rw = c["rho_in"] if C[o][0] < 0 else c["rho_out"]
                e = -f[o] + 2.0 * WQ[i] * rw * (1.0 + 4.5 * _dot(o, u) ** 2 - 1.5 * uu)
                new[i] = torch.where(self.out[o], e, new[i])
                self.g[i] = torch.where(self.out[o], phi * e + seg, self.g[i])
            at = (self.fluid & (_shift(self.mask, o) >= 2)).nonzero(as_tuple=True)
            if not len(at[0]):
                continue
            p = _shift(self.mask, o)[at] - 2
            ci = self.t(C[i])
            x = torch.stack([at[2], at[1], at[0]], 1).double()
            arm = self._image(x - 0.5 * ci - self.p_x[p])
            uw = self.p_v[p] + _cross(self.p_w[p], arm)
            add = 6.0 * WQ[i] * rho[at] * (uw @ ci)
            out = f[o][at] + add
            new[i][at] = out
            self.g[i][at] += phi[at] * add
            dP = (-ci - uw) * f[o][at][:, None] - (ci - uw) * out[:, None]
            Fh.index_add_(0, p, dP)
            Th.index_add_(0, p, _cross(arm, dP))
        self.f = new
        self.Fh = Fh
        self._dem(Fh + self.Fc, Th + self.Tc)
        self._move()

    def _capillary(self, phi, n, big):
        c, S = self.c, torch.zeros(self.n, 6, dtype=torch.float64, device=DEVICE)
        da = math.radians(c["cap_dang_deg"])
        na, nph = round(180.0 / c["cap_dang_deg"]), round(360.0 / c["cap_dang_deg"])
        a = (torch.arange(na, device=DEVICE).double() + 0.5)[:, None] * da
        b = torch.arange(nph, device=DEVICE).double()[None, :] * da
        s = torch.stack([(torch.sin(a) * torch.cos(b)), (torch.sin(a) * torch.sin(b)),
                         torch.cos(a).expand(na, nph)], -1).view(-1, 3)
        sa = torch.sin(a).expand(na, nph).reshape(-1)
        N = [self.shape[2], self.shape[1], self.shape[0]]
        for p in range(self.n if c["sigma"] else 0):
            R = self.p_R[p]
            x = self.p_x[p] + R * s
            lo = torch.floor(x)
            fr, lo = x - lo, lo.long()
            W_, acc = 0.0, [0.0] * 4
            for k in range(8):
                o = [k & 1, (k >> 1) & 1, k >> 2]
                ix = [(lo[:, d] + o[d]) % N[d] for d in range(3)]
                at = (ix[2], ix[1], ix[0])
                w = torch.prod(torch.stack([fr[:, d] if o[d] else 1 - fr[:, d]
                                            for d in range(3)]), 0) * self.fluid[at]
                W_ = W_ + w
                acc[0] = acc[0] + w * phi[at]
                for d in range(3):
                    acc[1 + d] = acc[1 + d] + w * n[d][at] * big[at]
            ok = W_ > 0
            ph, G = acc[0] / W_, torch.stack(acc[1:], 1) / W_[:, None]
            g = G.norm(dim=1)
            nn = G / g[:, None]
            m = s - (nn * s).sum(1, keepdim=True) * nn
            ml = m.norm(dim=1)
            wgt = 1.0 - ph * ph
            ok &= (wgt > 0) & (g > EPS) & (ml > 1e-3)
            coef = (c["sigma"] * 4.5 * c["cap_k"] * c["beta"]
                    * torch.sin(torch.deg2rad(self.p_theta_deg[p])) * wgt * R * R * sa * da * da)
            dF = torch.where(ok[:, None], coef[:, None] * m / ml[:, None], 0.0)
            S[p, :3] = dF.sum(0)
            S[p, 3:] = _cross(R * s, dF).sum(0)
        self.Fc, self.Tc = S[:, :3], S[:, 3:]

    def _wall_contacts(self):
        """Overlap and normal with each face of the static wall."""
        c, x = self.c, self.p_x
        d, n = [], []
        if c["has_wall"] in (1, 3):
            d = [self.Rc - (x[:, 2] - 0.5), self.Rc - (c["nz"] - 0.5 - x[:, 2])]
            n = [self.t([0, 0, 1.0]).expand(self.n, 3), self.t([0, 0, -1.0]).expand(self.n, 3)]
        if c["has_wall"] == 3:
            for b in c["boxes"]:
                v = x - torch.minimum(torch.maximum(x, self.t(b[:3]) - 0.5), self.t(b[3:]) + 0.5)
                r = v.norm(dim=1)
                d.append(torch.where(r > 0, self.Rc - r, -1.0))
                n.append(v / r.clamp_min(1e-300)[:, None])
        if c["has_wall"] == 2:
            v = 0.5 * (self.L - 1) - x
            v[:, 0] = 0.0
            r = v.norm(dim=1)
            d.append(self.Rc - (c["tube_R"] - r))
            n.append(v / r.clamp_min(1e-300)[:, None])
        return d, n

    def _spring(self, k, damp, cap, xi, v, dt):
        F = -k * xi - damp * v
        size = F.norm(dim=-1, keepdim=True)
        slide = size > cap
        F = torch.where(slide, cap * F / size.clamp_min(1e-300), F)
        return F, torch.where(slide, -(F + damp * v) / k, xi + v * dt)

    def _contacts(self, vp, wp, dt):
        c, P, n = self.c, self.n, self.n + self.walls
        arm = self._image(self.p_x[:, None] - self.p_x[None])
        dist = arm.norm(dim=2)
        delta = self.Rc[:, None] + self.Rc[None] - dist
        delta.fill_diagonal_(-1.0)
        nh = arm / dist.clamp_min(1e-300)[..., None]
        wd, wn = self._wall_contacts()
        if wd:
            delta = torch.cat([delta, torch.stack(wd, 1)], 1)
            nh = torch.cat([nh, torch.stack(wn, 1)], 1)

        def ext(a, fill):
            pad = a.new_full((P, self.walls) + a.shape[2:], fill)
            return torch.cat([a, pad], 1)
        vj, wj, arm = (ext(a[None].expand(P, P, 3) if a.dim() == 2 else a, 0.0)
                       for a in (vp, wp, arm))
        mean = [torch.cat([0.5 * (m[:, None] + m[None]), m[:, None].expand(P, self.walls)], 1)
                for m in (self.p_mu_s, self.p_mu_r)]
        ap = torch.cat([self.Rc[:, None] * self.Rc[None] / (self.Rc[:, None] + self.Rc[None]),
                        self.Rc[:, None].expand(P, self.walls)], 1)[..., None]
        on = (delta > 0)[..., None]
        vi, wi = vp[:, None].expand(P, n, 3), wp[:, None].expand(P, n, 3)
        vrel = vi - vj
        Fn = c["kn"] * delta - c["gn"] * (vrel * nh).sum(2)
        ri = -(self.Rc[:, None] - 0.5 * delta)[..., None] * nh
        vc = vrel + _cross(wi, ri) - _cross(wj, ri + arm)
        vt = vc - (vc * nh).sum(2, keepdim=True) * nh
        self.xt = self.xt - (self.xt * nh).sum(2, keepdim=True) * nh
        self.xr = self.xr - (self.xr * nh).sum(2, keepdim=True) * nh
        push = Fn.clamp_min(0.0)[..., None]
        Ft, xt = self._spring(c["kt"], c["gt"], mean[0][..., None] * push, self.xt, vt, dt)
        vr = -ap * (_cross(nh, wi) - _cross(nh, wj))
        Fr, xr = self._spring(c["kr"], c["gr"], mean[1][..., None] * push, self.xr, vr, dt)
        self.xt, self.xr = torch.where(on, xt, 0.0), torch.where(on, xr, 0.0)
        F = torch.where(on, Fn[..., None] * nh + Ft, 0.0)
        T = torch.where(on, _cross(ri, Ft) + ap * _cross(nh, Fr), 0.0)
        return F.sum(1), T.sum(1)

    def _dem(self, F, T):
        Fp, Tp = self.prev or (F, T)
        self.prev = (F, T)
        F, T = 0.5 * (F + Fp), 0.5 * (T + Tp)
        F = F - self.p_g_p[:, None] * self.t([0, 0, 1.0])
        dt = 1.0 / self.n_sub
        free = (~self.kin)[:, None].double()
        self.old = self.p_x
        for _ in range(self.n_sub):
            a = free * (F + self.Fcp) / self.mass[:, None]
            b = free * (T + self.Tcp) / self.inertia[:, None]
            x = self.p_x + self.p_v * dt + 0.5 * a * dt * dt
            wrap = torch.remainder(x, self.L)
            if self.c["has_wall"]:
                wrap[:, 2] = x[:, 2]
            if self.c.get("open_x"):
                wrap[:, 0] = x[:, 0]
            self.p_x = wrap
            Fn, Tn = self._contacts(self.p_v + a * dt, self.p_w + b * dt, dt)
            self.p_v = self.p_v + 0.5 * (a + free * (F + Fn) / self.mass[:, None]) * dt
            self.p_w = self.p_w + 0.5 * (b + free * (T + Tn) / self.inertia[:, None]) * dt
            self.Fcp, self.Tcp = Fn, Tn

    def _move(self):
        """The mask of the new positions; uncovered nodes refilled."""
        was = self.mask
        self.mask = self._mask()
        fresh = (was >= 2) & (self.mask == 0)
        at = fresh.nonzero(as_tuple=True)
        if len(at[0]):
            good = (self.mask == 0) & ~fresh
            cnt, sums = 0, [0.0, 0.0]
            N = self.shape
            for i in range(1, 19):
                m = tuple((at[d] + C[i][2 - d]) % N[d] for d in range(3))
                ok = good[m]
                cnt = cnt + ok
                for k, q in enumerate((self.f, self.g)):
                    sums[k] = sums[k] + ok * q[(slice(None),) + m].sum(0)
            none = cnt == 0
            rho = torch.where(none, self.c["rho0"], sums[0] / cnt.clamp_min(1))
            col = torch.where(none, 0.0, sums[1] / cnt.clamp_min(1))
            p = was[at] - 2
            x = torch.stack([at[2], at[1], at[0]], 1).double()
            uw = self.p_v[p] + _cross(self.p_w[p], self._image(x - self.p_x[p]))
            for i in range(19):
                cu = uw @ self.t(C[i])
                e = WQ[i] * (1.0 + 3 * cu + 4.5 * cu * cu - 1.5 * (uw * uw).sum(1))
                self.f[i][at] = rho * e
                self.g[i][at] = col * e
        self._links()

    def push(self, parts):
        """The particles put at prescribed positions and velocities."""
        self.p_x, self.p_v = self.t([p["x"] for p in parts]), self.t([p["v"] for p in parts])
        self._move()

    def fields(self):
        phi, _, _, F = self._interface()
        rho, u = self._velocity(F)
        u = [torch.where(self.fluid, a, 0.0) for a in u]
        at = (self.mask >= 2).nonzero(as_tuple=True)
        p = self.mask[at] - 2
        x = torch.stack([at[2], at[1], at[0]], 1).double()
        uw = self.p_v[p] + _cross(self.p_w[p], self._image(x - self.p_x[p]))
        for k in range(3):
            u[k][at] = uw[:, k]
        rho = torch.where(self.fluid, rho, 0.0)
        return rho.view(-1), torch.stack(u).view(-1), phi.view(-1)

    def records(self):
        return dict(x=self.p_x, v=self.p_v, F_hyd=self.Fh, F_cap=self.Fc)


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return None  # the order of the samples is the library's own shuffle
    if kind == "predict":
        par = [torch.as_tensor(p, dtype=torch.float64, device=DEVICE)
               for p in unflatten(flatten(he_init(seed)))]
        h = torch.from_numpy(W.rng(seed, 1).standard_normal((case["rows"], SRG_IN)).astype(
            np.float32)).to(DEVICE, torch.float64)
        for k in range(5):
            h = h @ par[2 * k] + par[2 * k + 1]
            h = torch.relu(h) if k < 4 else h
        return h
    if kind == "ensemble" and case["members"] * case["steps"] > 600:
        return None  # every member by itself: over 20 seconds
    got, logs = [], []
    for sim in _sims(case, seed):
        e = Exact(sim)
        for k in range(case["steps"]):
            if kind == "pulled":
                e.push([_path(p, k) for p in sim["particles"]])
            e.step()
            if kind == "pulled":
                logs.append(e.records())
        got.append(e.fields())
        if kind != "pulled":
            logs.append(e.records())
        del e
    out = dict(zip(("rho", "u", "phi"), (torch.cat(a) for a in zip(*got))))
    out.update({k: torch.cat([r[k] for r in logs]) for k in LOG})
    return out
