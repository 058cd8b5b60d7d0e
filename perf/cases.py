"""The work that programs have this framework do, as cases to measure.

  listed()             the cases
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  a running simulation, or a network and its data, on the GPU
  run(state)           one pass through the public entry points, and its outputs
  exact(case, seed)    the outputs of the first pass, in 64 bits from plain torch
  work(case)           bytes and operations one pass cannot do without

Two kinds of case.  "box" steps a suspension: one box, or an ensemble of
boxes, of any lattice, storage and option, from fluid at rest with particles
that already move, then reads the particles' state (and the fields, where a
program writes snapshots).  "mlp" runs the closure network forward, its
gradient over a data set, or a stretch of training.

exact() is the method restated on dense arrays in FP64 (collision, boundary
sites, particle update, internal sites, propagation), with no code of the
package in it.
"""
import math

import numpy as np
import torch

from paper_1105_2904_amd import lbm
from paper_1105_2904_amd import workloads as wl


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------
def _box(name, **kw):
    c = {"name": name, "kind": "box", "q": 19, "nx": 64, "ny": 64, "nz": 1, "boxes": 1, "tau": 0.7, "storage": "fp32",
         "particles": 1, "rmin": 6.0, "rmax": 6.0, "ratio": 1.5, "gravity": 1e-5, "kinematic": False, "walls": 0,
         "aa": False, "graph": 0, "width": -1, "cap": 0, "closure": False, "steps": 10, "fields": False}
    c.update(kw)
    return c


def _mlp(name, what, **kw):
    c = {"name": name, "kind": "mlp", "what": what, "rows": 4096}
    c.update(kw)
    return c


def listed():
    return [
        # one disk dragged through a small FP64 box: the paper's drag runs, the
        # smallest problem and all launch latency
        _box("disk-64-fp64", q=9, nx=64, ny=64, tau=0.8, storage="fp64", rmin=8.0, rmax=8.0, gravity=0.0,
             kinematic=True, steps=20),
        # held-out pair boxes with the near-contact closure on, the forces read
        # after every step: the shortest call a program makes
        _box("pairs-closure-fp32", q=9, nx=52, ny=76, boxes=16, particles=2, rmin=6.0, rmax=12.0, closure=True, steps=1),
        # the same pairs at four times the resolution, where the training forces
        # come from: balls too large for the per-particle ownership grids
        _box("pairs-refined-fp32", q=9, nx=208, ny=304, boxes=32, particles=2, rmin=24.0, rmax=48.0, gravity=1e-7,
             steps=16),
        # one 2D suspension, replayed from step graphs: cache resident
        _box("disks-1024-fp32", q=9, nx=1024, ny=1024, particles=200, rmin=10.0, rmax=10.0, graph=20, steps=40),
        # an ensemble of uneven 2D boxes, one launch per kernel for all of them
        _box("ensemble-64-fp32", q=9, nx=128, ny=512, boxes=64, particles=80, rmin=6.0, rmax=12.0, graph=20, width=256,
             steps=20),
        # a sphere settling in a closed box (100 sites to a row), FP64, with a
        # snapshot of the fields after the steps
        _box("settling-walls-fp64", nx=100, ny=100, nz=160, tau=0.9, storage="fp64", rmin=7.5, rmax=7.5, ratio=1.1546,
             gravity=1.18e-3, walls=7, steps=50, fields=True),
        # the headline suspension at its tuned launch, 32- and 16-bit storage
        _box("spheres-256-fp32", nx=256, ny=256, nz=256, tau=0.6, particles=500, ratio=1.2, gravity=1e-6, width=256,
             cap=5),
        _box("spheres-256-fp16", nx=256, ny=256, nz=256, tau=0.6, particles=500, ratio=1.2, gravity=1e-6,
             storage="fp16", width=0, cap=5),
        # an odd box at the default launch with the smallest state there is:
        # 16-bit storage in one array
        _box("spheres-odd-bf16-aa", nx=191, ny=157, nz=173, tau=0.65, particles=120, rmin=4.0, rmax=7.0, ratio=1.2,
             gravity=1e-6, storage="bf16", aa=True),
        # the closure network: inference over many pairs, the gradient over a
        # data set, and a stretch of training
        _mlp("mlp-forward-4m", "forward", rows=4194304),
        _mlp("mlp-gradient-44672", "gradient", rows=44672),
        _mlp("mlp-train-500", "train", rows=44672, batch=256, steps=500),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _fits(c):
    """Most particles per box that random placement reaches easily."""
    n = [c["nx"], c["ny"], c["nz"]] if c["boxes"] == 1 else [c["nx"]] * 2 + [1]
    inner = [m - (2 * int(4.0 + c["rmax"]) if (c["walls"] >> a) & 1 else 0) for a, m in enumerate(n)]
    r = c["rmax"] + 1.0
    if c["q"] == 9:
        return int(0.3 * inner[0] * inner[1] / (math.pi * r * r))
    return int(0.18 * inner[0] * inner[1] * inner[2] / (4.0 / 3.0 * math.pi * r ** 3))


def draw(rng):
    u = rng.random()
    if u < 0.25:
        what = rng.choice(["forward", "gradient", "train"])
        if what == "forward":
            return dict(_mlp("", what, rows=_log_int(rng, 1, 4194304)))
        if what == "gradient":
            return dict(_mlp("", what, rows=_log_int(rng, 16, 131072)))
        return dict(_mlp("", what, rows=_log_int(rng, 300, 65536), batch=64 * rng.randint(1, 8), steps=_log_int(rng, 20, 400)))
    storage = rng.choice(["fp32", "fp32", "fp32", "fp64", "fp16", "bf16"])
    aa = rng.random() < 0.2
    tau = round(rng.uniform(0.6, 1.0), 3)
    graph = rng.choice([0, 0, 10])
    if u < 0.45:  # ensembles of uneven boxes
        small = rng.random() < 0.5
        c = _box("", q=9, boxes=_log_int(rng, 4, 64), nx=rng.randint(52, 80) if small else rng.randint(128, 200),
                 ny=rng.randint(81, 120) if small else rng.randint(201, 512), rmin=6.0, rmax=12.0,
                 particles=2 if small else rng.randint(10, 80), closure=small and rng.random() < 0.5)
    elif u < 0.55:  # large disks
        c = _box("", q=9, boxes=_log_int(rng, 2, 32), nx=rng.randint(200, 230), ny=rng.randint(231, 320), particles=2,
                 rmin=24.0, rmax=48.0, gravity=1e-7)
        aa = False
    elif u < 0.75:  # one 2D box
        r = round(rng.uniform(3.0, 12.0), 2)
        c = _box("", q=9, nx=_log_int(rng, 48, 1200), ny=_log_int(rng, 48, 1200), rmin=r, rmax=r,
                 walls=rng.choice([0, 0, 2, 3]))
        c["particles"] = max(1, min(_fits(c), _log_int(rng, 1, 300)))
    else:  # one 3D box
        r = round(rng.uniform(3.0, 8.0), 2)
        c = _box("", nx=_log_int(rng, 40, 250), ny=_log_int(rng, 40, 250), nz=_log_int(rng, 40, 250), rmin=r, rmax=r,
                 ratio=1.2, gravity=1e-6, walls=rng.choice([0, 0, 0, 7]))
        c["particles"] = max(1, min(_fits(c), _log_int(rng, 1, 500)))
    c.update(storage=storage, aa=aa, tau=tau, graph=graph, steps=graph if graph else rng.randint(1, 10))
    sites = _sites(c)
    c["fields"] = sites <= 1 << 20 and rng.random() < 0.4
    return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _dims(c):
    """Box sizes: one nx x ny x nz box, or square boxes of side nx..ny (the
    sides belong to the case, not to the seed)."""
    if c["boxes"] == 1:
        return [(c["nx"], c["ny"], c["nz"])]
    rng = wl.SplitMix64(1000 + c["boxes"])
    out = []
    for _ in range(c["boxes"]):
        n = rng.randint(c["nx"], c["ny"])
        out.append((n, n, 1))
    return out


def _particles(c, seed):
    """Per box: centres, velocities, spins, radii, masses and inertias.  Radii and
    counts belong to the case, positions and velocities to the seed."""
    dim = 2 if c["q"] == 9 else 3
    shape = wl.SplitMix64(7 + c["boxes"])
    out = []
    for b, box in enumerate(_dims(c)):
        n = c["particles"] if c["boxes"] == 1 else (2 if c["particles"] == 2 else shape.randint(10, c["particles"]))
        radii = np.array([c["rmin"] + (c["rmax"] - c["rmin"]) * shape.uniform() for _ in range(n)])
        if c["boxes"] > 1 and c["particles"] != 2:  # drop the last ones above an area fraction of 1/4
            keep = n
            while keep > 1 and np.pi * (radii[:keep] ** 2).sum() > 0.25 * box[0] * box[1]:
                keep -= 1
            radii, n = radii[:keep], keep
        key = seed * 1009 + b
        rng = wl.SplitMix64(key)
        if c["particles"] == 2 and c["boxes"] > 1:
            # a near-contact pair about the box's centre, on a random axis
            th = 2.0 * math.pi * rng.uniform()
            gap = (0.3 + 1.5 * rng.uniform()) * c["rmin"] / 6.0
            e = np.array([math.cos(th), math.sin(th)])
            m = np.array([box[0] / 2.0 + rng.uniform() - 0.5, box[1] / 2.0 + rng.uniform() - 0.5])
            x = np.zeros((2, 3))
            x[0, :2] = m - e * (radii[0] + 0.5 * gap)
            x[1, :2] = m + e * (radii[1] + 0.5 * gap)
        elif c["walls"]:
            # inside the walls: random placement in the space between them
            pad = [4.0 if (c["walls"] >> a) & 1 else 0.0 for a in range(3)]
            inner = tuple(box[a] - 2 * int(pad[a] + c["rmax"]) if pad[a] else box[a] for a in range(3))
            x = wl.place_particles(inner if dim == 3 else (inner[0], inner[1], 1), radii, key)
            for a in range(dim):
                x[:, a] += int(pad[a] + c["rmax"]) if pad[a] else 0.0
        else:
            x = wl.place_particles(box, radii, key)
        m, inertia = wl.solid_body(dim, radii, c["ratio"])
        if c["kinematic"]:
            m, inertia = np.full(n, np.inf), np.full(n, np.inf)
        u = wl.seeded_velocities(n, dim, 0.01, key + 1)
        om = np.zeros((n, 3))
        om[:, 2] = [1e-3 * (2.0 * rng.uniform() - 1.0) for _ in range(n)]
        out.append({"x": x, "u": u, "omega": om, "radius": radii, "mass": np.asarray(m, dtype=np.float64),
                    "inertia": np.asarray(inertia, dtype=np.float64)})
    return out


def _gravity(c):
    return (0.0, -c["gravity"], 0.0) if c["q"] == 9 else (0.0, 0.0, -c["gravity"])


def _network(seed):
    """Network parameters: Glorot weights and small biases, float32 values."""
    p = wl.mlp_init(seed % 100003).copy()
    rng = np.random.Generator(np.random.PCG64(seed))
    b = p == 0.0
    p[b] = rng.uniform(-0.1, 0.1, size=int(b.sum()))
    return p.astype(np.float32)


def _rows(c, seed):
    """Closure inputs (gap, radii, normal, offset, tau) and targets, float32,
    on the GPU."""
    n = c["rows"]
    g = torch.Generator(device="cuda").manual_seed(seed)
    v = torch.rand((n, 6), device="cuda", generator=g)
    x = torch.empty((n, 8), device="cuda")
    x[:, 0] = 0.25 + 1.75 * v[:, 0]
    x[:, 1:3] = 2.0 * v[:, 1:3] - 1.0
    x[:, 3] = torch.cos(2.0 * math.pi * v[:, 3])
    x[:, 4] = torch.sin(2.0 * math.pi * v[:, 3])
    x[:, 5:7] = v[:, 4:6] - 0.5
    x[:, 7] = 0.0
    t = torch.stack([1.0 / (0.5 + x[:, 0]) - 0.8 + 0.3 * x[:, 3] * x[:, 5], 0.5 * x[:, 4] * x[:, 6] + 0.2 * x[:, 1]], dim=1)
    t = t + 0.1 * (torch.rand((n, 2), device="cuda", generator=g) - 0.5)
    return x.contiguous(), t.contiguous()


def prepare(case, seed):
    c = case
    if c["kind"] == "mlp":
        x, t = _rows(c, seed)
        p = torch.tensor(_network(seed), device="cuda")
        s = {"case": c, "p": p, "x": x, "t": t}
        if c["what"] == "train":
            s.update(m=torch.zeros_like(p), v=torch.zeros_like(p), done=0)
        return s
    dims, parts = _dims(c), _particles(c, seed)
    n = sum(len(p["radius"]) for p in parts)
    kw = dict(tau=c["tau"], gravity=_gravity(c), zero_net_force=not c["walls"], storage=c["storage"], max_particles=n,
              max_radius=float(max(p["radius"].max() for p in parts)), walls=c["walls"], aa=c["aa"])
    if c["boxes"] == 1:
        sim = lbm.Simulation(c["q"], *dims[0], **kw)
    else:
        sim = lbm.Simulation(c["q"], 1, 1, 1, boxes=dims, **kw)
    for b, p in enumerate(parts):
        sim.add_particles(p["x"], u=p["u"], omega=p["omega"], radius=p["radius"], mass=p["mass"], inertia=p["inertia"],
                          box=b)
    if c["width"] >= 0:
        sim.set_sweep_config(c["width"], 0, c["cap"])
    if c["closure"]:
        sim.set_closure(torch.tensor(_network(seed), device="cuda"), 2.0)
    if c["graph"]:
        sim.set_graph(c["graph"])
    return {"case": c, "sim": sim}


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def run(state):
    c = state["case"]
    if c["kind"] == "mlp":
        if c["what"] == "forward":
            return {"y": lbm.mlp_forward(state["p"], state["x"])}
        if c["what"] == "gradient":
            loss, g = lbm.mlp_gradient(state["p"], state["x"], state["t"])
            return {"grad": g, "loss": loss}
        losses = lbm.mlp_train(state["p"], state["m"], state["v"], state["x"], state["t"], batch=c["batch"],
                               steps=c["steps"], step0=state["done"], lr=2e-3)
        state["done"] += c["steps"]
        return {"losses": losses, "p": state["p"], "m": state["m"], "v": state["v"]}
    sim = state["sim"]
    sim.step(c["steps"])
    F, T, x, u, omega = sim.forces()
    out = {"F": F, "T": T, "x": x, "u": u, "omega": omega}
    if c["fields"]:
        out["rho"], out["vel"], out["owner"] = sim.fields()
    return out


def _sites(c):
    return sum(a * b * d for a, b, d in _dims(c))


def work(case):
    c = case
    if c["kind"] == "mlp":
        fwd, params = 2 * (8 * 64 + 64 * 64 + 64 * 2), 4866
        if c["what"] == "forward":
            return {"bytes": c["rows"] * 40 + 4 * params, "flops": c["rows"] * fwd}
        if c["what"] == "gradient":
            return {"bytes": c["rows"] * 40 + 8 * params, "flops": 3 * c["rows"] * fwd}
        rows = c["batch"] * c["steps"]
        return {"bytes": min(rows, c["rows"]) * 40 + 24 * params, "flops": 3 * rows * fwd}
    # every population read once and written once a step; about 12 operations
    # per population and 30 per site in the collision
    size = {"fp64": 8, "fp32": 4, "fp16": 2, "bf16": 2}[c["storage"]]
    n = _sites(c)
    b = 2.0 * c["q"] * size * n * c["steps"]
    if c["fields"]:
        b += (c["q"] * size + 36.0) * n
    return {"bytes": b, "flops": (12.0 * c["q"] + 30.0) * n * c["steps"]}


# ---------------------------------------------------------------------------
# The same passes in 64 bits
# ---------------------------------------------------------------------------
_C9 = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (-1, 0, 0), (0, -1, 0), (1, 1, 0), (-1, 1, 0), (-1, -1, 0), (1, -1, 0)]
_C19 = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 0), (-1, -1, 0),
        (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1), (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1),
        (0, -1, 1)]


def _template(q, r, phi):
    """Ball sites by offset: boundary sites (linked to the outside), then
    internal ones (linked to a boundary site)."""
    C = _C9 if q == 9 else _C19
    R = int(math.ceil(r)) + 1
    g = np.arange(-R - 1, R + 2)
    Z, Y, X = np.meshgrid(g if q == 19 else np.array([0]), g, g, indexing="ij")
    inside = (X - phi[0]) ** 2 + (Y - phi[1]) ** 2 + (Z - phi[2]) ** 2 <= r * r

    def at(a, c):
        return np.roll(a, (-c[2], -c[1], -c[0]), axis=(0, 1, 2))

    bs = inside & np.any([~at(inside, c) for c in C[1:]], axis=0)
    ins = inside & ~bs & np.any([at(bs, c) for c in C[1:]], axis=0)
    both = [np.stack([X[s], Y[s], Z[s]], axis=1) for s in (bs, ins)]
    return np.concatenate(both), np.concatenate([np.ones(len(both[0]), int), np.full(len(both[1]), 2)])


def _network64(p, x):
    w1, b1 = p[:512].reshape(8, 64), p[512:576]
    w2, b2 = p[576:4672].reshape(64, 64), p[4672:4736]
    w3, b3 = p[4736:4864].reshape(64, 2), p[4864:]
    return torch.tanh(torch.tanh(x @ w1 + b1) @ w2 + b2) @ w3 + b3


class _Box64:
    """One box of the method on dense arrays, FP64."""

    def __init__(self, c, box, parts, net, dev):
        self.c, self.dev, self.net = c, dev, net
        self.n = np.array(box)
        self.N = int(np.prod(box))
        self.C = _C9 if c["q"] == 9 else _C19
        self.dim = 2 if c["q"] == 9 else 3
        rest = {9: 4 / 9, 19: 1 / 3}[c["q"]]
        face = {9: 1 / 9, 19: 1 / 18}[c["q"]]
        self.w = [rest if sum(map(abs, k)) == 0 else face if sum(map(abs, k)) == 1 else 1 / 36 for k in self.C]
        self.x, self.u, self.om = parts["x"].copy(), parts["u"].copy(), parts["omega"].copy()
        if self.dim == 2:
            self.x[:, 2] = 0.0
        self.x0, self.r, self.m, self.I = self.x.copy(), parts["radius"], parts["mass"], parts["inertia"]
        self.b0 = np.floor(self.x + 0.5).astype(int)
        phi = self.x - self.b0
        self.k = np.zeros_like(self.b0)
        off, kind, pid = [], [], []
        for j in range(len(self.r)):
            o, t = _template(c["q"], self.r[j], phi[j])
            off.append(o)
            kind.append(t)
            pid.append(np.full(len(o), j))
        t64 = dict(device=dev, dtype=torch.float64)
        self.off = torch.tensor(np.concatenate(off), device=dev)
        self.kind = torch.tensor(np.concatenate(kind), device=dev)
        self.pid = torch.tensor(np.concatenate(pid), device=dev)
        self.arm = self.off.to(torch.float64) - torch.tensor(phi, **t64)[self.pid]
        V = np.pi * self.r ** 2 if self.dim == 2 else 4.0 / 3.0 * np.pi * self.r ** 3
        heavy = np.where(np.isinf(self.m), 0.0, self.m - V)
        self.fext = heavy[:, None] * np.array(_gravity(c))
        self.fb = -self.fext.sum(axis=0) / self.N if not c["walls"] else np.zeros(3)
        shape = tuple(int(v) for v in self.n[::-1])
        self.g = torch.zeros((c["q"],) + shape, **t64)
        self.wall = torch.zeros(shape, dtype=torch.bool, device=dev)
        for a in range(3):
            if (c["walls"] >> a) & 1:
                edge = torch.arange(int(self.n[a]), device=dev)
                edge = (edge < 2) | (edge >= int(self.n[a]) - 2)
                self.wall |= edge.reshape([-1 if 2 - a == d else 1 for d in range(3)])
        self.F = self.T = np.zeros_like(self.x)

    def _eq(self, i, dr, ux, uy, uz):
        cx, cy, cz = self.C[i]
        cu = cx * ux + cy * uy + cz * uz
        return self.w[i] * (dr + (1.0 + dr) * (3.0 * cu + 4.5 * cu * cu - 1.5 * (ux * ux + uy * uy + uz * uz)))

    def _moments(self, g):
        dr = g.sum(dim=0)
        j = [torch.zeros_like(dr) for _ in range(3)]
        for i, c in enumerate(self.C):
            for a in range(3):
                if c[a]:
                    j[a] += c[a] * g[i]
        return dr, j

    def _owned(self):
        """Sites of the entries, and which entries own theirs (lowest particle;
        none on walls)."""
        n = torch.tensor(self.n, device=self.dev)
        at = (self.off + torch.tensor(self.b0 + self.k, device=self.dev)[self.pid]) % n
        s = at[:, 0] + n[0] * (at[:, 1] + n[1] * at[:, 2])
        e = torch.arange(len(s), device=self.dev)
        first = torch.full((self.N,), len(s), device=self.dev).scatter_reduce(0, s, e, "amin")
        return s, (first[s] == e) & ~self.wall.reshape(-1)[s]

    def _rigid(self, sel):
        t = lambda v: torch.tensor(v, device=self.dev)[self.pid[sel]]
        return t(self.u) + torch.linalg.cross(t(self.om), self.arm[sel])

    def _impose(self, s, dr, v):
        flat = self.g.reshape(len(self.C), -1)
        for i in range(len(self.C)):
            flat[i, s] = self._eq(i, dr, v[:, 0], v[:, 1], v[:, 2])

    def _image(self, d):
        d = d.copy()
        L = self.n[:self.dim].astype(float)
        d[..., :self.dim] -= L * np.floor(d[..., :self.dim] / L + 0.5)
        return d

    def _closure(self):
        fc = np.zeros_like(self.x)
        mu = (self.c["tau"] - 0.5) / 3.0
        for i in range(len(self.r)):
            for j in range(i + 1, len(self.r)):
                d = self._image(self.x[j] - self.x[i])
                dist = math.sqrt((d * d).sum())
                h = dist - self.r[i] - self.r[j]
                if not h < 2.0:
                    continue
                e = d / dist
                mid = self.x[i] + e * (self.r[i] + 0.5 * h)
                o = mid - np.floor(mid + 0.5)
                f = [h, (self.r[i] - 9) / 3, (self.r[j] - 9) / 3, e[0], e[1], o[0], o[1], (self.c["tau"] - 0.7) / 0.1]
                a = _network64(self.net, torch.tensor(f, device=self.dev, dtype=torch.float64)).cpu().numpy()
                U = ((self.u[i] - self.u[j]) * e).sum()
                f = mu * U * (a[0] * e + a[1] * np.array([-e[1], e[0], 0.0]))
                fc[i] += f
                fc[j] -= f
        return fc

    def _collide(self):
        close = np.linalg.norm(self._image(self.x[None] - self.x[:, None]), axis=2) <= self.r[None] + self.r[:, None] + 1
        for i, j in np.argwhere(np.triu(close, 1)):
            A, B = np.isinf(self.m[i]), np.isinf(self.m[j])
            d = self._image(self.x[j] + self.u[j] - self.x[i] - self.u[i])
            dist = math.sqrt((d * d).sum())
            if (A and B) or dist > self.r[i] + self.r[j] or dist == 0.0:
                continue
            e = d / dist
            if not ((self.u[j] - self.u[i]) * e).sum() < 0.0:
                continue
            W = self.u[i].copy() if A else self.u[j].copy() if B else (
                (self.m[i] * self.u[i] + self.m[j] * self.u[j]) / (self.m[i] + self.m[j]))
            for q in (i, j):
                v = self.u[q] - W
                self.u[q] = W + v - 2.0 * (v * e).sum() * e
        for a in range(self.dim):
            if (self.c["walls"] >> a) & 1:
                x = self.x[:, a] + self.u[:, a]
                hit = ((x - self.r <= 1.0) & (self.u[:, a] < 0)) | ((x + self.r >= self.n[a] - 2) & (self.u[:, a] > 0))
                self.u[hit & ~np.isinf(self.m), a] *= -1.0

    def step(self):
        om = 1.0 / self.c["tau"]
        dr, j = self._moments(self.g)
        v = [k / (1.0 + dr) for k in j]
        for i in range(len(self.C)):
            f = 3.0 * self.w[i] * float(np.dot(self.C[i], self.fb))
            self.g[i] += om * (self._eq(i, dr, *v) - self.g[i]) + f
        # boundary sites and the momentum they exchange
        s, own = self._owned()
        sel = own & (self.kind == 1)
        sb, vb = s[sel], self._rigid(sel)
        db, jb = self._moments(self.g.reshape(len(self.C), -1)[:, sb])
        dp = (1.0 + db)[:, None] * vb - torch.stack(jb, dim=1)
        dl = torch.linalg.cross(self.arm[sel], dp)
        sums = torch.zeros((len(self.r), 6), device=self.dev, dtype=torch.float64)
        sums.index_add_(0, self.pid[sel], torch.cat([dp, dl], dim=1))
        sums = sums.cpu().numpy()
        self._impose(sb, db, vb)
        if self.c["walls"]:
            for i in range(len(self.C)):
                self.g[i] = torch.where(self.wall, self.w[i] * dr, self.g[i])
        # particles
        fc = self._closure() if self.c["closure"] else 0.0
        self.F, self.T = -sums[:, :3] + fc, -sums[:, 3:]
        free = ~np.isinf(self.m)
        self.u[free] += ((self.fext + self.F) / self.m[:, None])[free]
        self.om[free] += (self.T / self.I[:, None])[free]
        self._collide()
        self.x += self.u
        self.k = np.floor(self.x - self.x0 + 0.5).astype(int)
        # internal sites at the new positions, propagation
        s, own = self._owned()
        sel = own & (self.kind == 2)
        self._impose(s[sel], self.g.reshape(len(self.C), -1)[:, s[sel]].sum(dim=0), self._rigid(sel))
        for i, c in enumerate(self.C):
            self.g[i] = torch.roll(self.g[i], (c[2], c[1], c[0]), dims=(0, 1, 2))

    def fields(self):
        dr, j = self._moments(self.g)
        s, own = self._owned()
        owner = torch.full((self.N,), -1, device=self.dev, dtype=torch.int32)
        owner[s[own]] = self.pid[own].to(torch.int32)
        return 1.0 + dr, torch.stack(j, dim=3) / (1.0 + dr)[..., None], owner.reshape(dr.shape)


def _mlp64(c, seed):
    dev = "cuda"
    x, t = _rows(c, seed)
    p = torch.tensor(_network(seed), device=dev).to(torch.float64)
    if c["what"] == "forward":
        return {"y": torch.cat([_network64(p, part.to(torch.float64)) for part in x.split(1 << 19)])}
    x, t = x.to(torch.float64), t.to(torch.float64)

    def loss_grad(q, a, b):
        q = q.detach().requires_grad_(True)
        loss = ((_network64(q, a) - b) ** 2).sum() / len(a)
        loss.backward()
        return loss.detach(), q.grad

    if c["what"] == "gradient":
        loss, g = loss_grad(p, x, t)
        return {"grad": g, "loss": loss.reshape(1)}
    m, v, losses = torch.zeros_like(p), torch.zeros_like(p), []
    for s in range(c["steps"]):
        at = (s * c["batch"] + torch.arange(c["batch"], device=dev)) % c["rows"]
        loss, g = loss_grad(p, x[at], t[at])
        losses.append(loss)
        m = 0.9 * m + 0.1 * g
        v = 0.999 * v + 0.001 * g * g
        p = p - 2e-3 * (m / (1 - 0.9 ** (s + 1))) / (torch.sqrt(v / (1 - 0.999 ** (s + 1))) + 1e-8)
    return {"losses": torch.stack(losses), "p": p, "m": m, "v": v}


def exact(case, seed):
    c = case
    if c["kind"] == "mlp":
        return _mlp64(c, seed)
    dev = "cuda"
    net = torch.tensor(_network(seed), device=dev).to(torch.float64) if c["closure"] else None
    boxes = [_Box64(c, d, p, net, dev) for d, p in zip(_dims(c), _particles(c, seed))]
    for b in boxes:
        for _ in range(c["steps"]):
            b.step()
    out = {k: np.concatenate([getattr(b, k) for b in boxes]) for k in ("F", "T", "x", "u")}
    out["omega"] = np.concatenate([b.om for b in boxes])
    if c["fields"]:
        rho, vel, owner, first = [], [], [], 0
        for b in boxes:  # particle ids run over the boxes
            r, v, o = b.fields()
            rho.append(r)
            vel.append(v)
            owner.append(torch.where(o >= 0, o + first, o))
            first += len(b.r)
        if len(boxes) > 1:
            rho, vel, owner = ([v.reshape((-1,) + v.shape[3:]) for v in k] for k in (rho, vel, owner))
        out["rho"], out["vel"], out["owner"] = torch.cat(rho), torch.cat(vel), torch.cat(owner)
    return out
